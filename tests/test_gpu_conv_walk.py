"""The sparse neighbour conv on the shapes its slot-walking kernel serves:
small active sets and channel counts the other conv kernels do not take, at
the edges of its 16- and 128-row workgroups, 32- and 64-column slices and
256-byte reduction phases (phases that hold several slots, k-steps that cross
a slot, a partial last phase), from a table and from coordinates (the same
bits), with and without bias and ReLU, against the oracle (Eqs. 4-5).  Every
input is seeded and synthetic.
"""
import numpy as np
import pytest
import torch

from oracle import shc_oracle as O
from paper_2608_09388_amd import binding as shc
from paper_2608_09388_amd import synth
from tests.gpu_util import TORCH, Compaction, assert_scaled_close, down, require_gpu, up

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("dtype,B,V,n,K,Cin,Cout", [
    ("f32", 1, 40, 1, 9, 16, 64),          # one row
    ("f32", 2, 60, 17, 9, 16, 16),         # a second block of one row, 4 slots a phase
    ("f32", 4, 655, 262, 9, 16, 64),       # the tiny layer
    ("f32", 3, 500, 129, 5, 48, 80),       # partial columns, phases across slots
    ("f32", 3, 900, 255, 9, 192, 64),      # three phases a slot
    ("f32", 6, 700, 1000, 32, 32, 48),     # 32 slots
    ("f32", 40, 655, 9000, 9, 16, 64),     # 128 x 32 workgroups, a ragged last one
    ("f32", 30, 655, 8321, 3, 144, 144),   # 128 x 32, K Cin past a phase
    ("f32", 40, 655, 17001, 9, 128, 128),  # split products, 256-row workgroups
    ("f32", 40, 900, 23000, 20, 48, 80),   # the same, 20 slots of 48 channels
    ("f32", 60, 655, 33500, 9, 128, 128),  # split products, 128-row workgroups
    ("f32", 90, 655, 50001, 3, 144, 80),   # the same, K Cin past a phase
    ("bf16", 1, 40, 15, 9, 16, 16),        # a k-step over two slots
    ("bf16", 3, 500, 128, 7, 48, 80),      # k-steps that cross slots
    ("bf16", 5, 655, 1000, 9, 64, 128),    # the encoder's widening layer
    ("bf16", 5, 655, 400, 9, 256, 256),    # 256 channels
    ("bf16", 4, 400, 700, 20, 80, 32),     # 20 slots, an odd multiple of 16
    ("bf16", 37, 1723, 19125, 7, 48, 80),  # 128 x 32
    ("bf16", 60, 655, 30001, 5, 32, 80),   # 128 x 64
])
def test_conv_walk_against_oracle(dev, dtype, B, V, n, K, Cin, Cout):
    rng = np.random.default_rng(B + V + 7 * n + 31 * K + Cin + Cout)
    nbr = rng.integers(-2, V + 2, size=(V, K)).astype(np.int32)   # some out of range: absent
    nbr[:, 0] = np.arange(V)
    m = np.zeros(B * V, dtype=np.uint8)
    m[rng.permutation(B * V)[:n]] = 1
    m = m.reshape(B, V)
    c = Compaction(m)
    assert c.run() == n
    S = synth.as_dtype(rng.standard_normal((n, Cin)).astype(np.float32), dtype)[1]
    W = synth.as_dtype((rng.standard_normal((K, Cin, Cout)) / np.sqrt(K * Cin))
                       .astype(np.float32), dtype)[1]
    bias = rng.standard_normal(Cout).astype(np.float32)
    coords, _, _, _ = O.compact(m)
    rows = np.unique(np.concatenate([np.arange(min(n, 150)), np.arange(max(0, n - 150), n),
                                     rng.choice(n, size=min(n, 300), replace=False)]))
    Sd, Wd, nd = up(S, dtype), up(W, dtype), up(nbr)
    table = torch.full((K * n,), -7, dtype=torch.int32, device=dev)
    shc.build_neighbor_table(c.coords, c.inv, n, B, V, nd, table)
    oob = np.where((nbr < 0) | (nbr >= V), -1, nbr)
    for b, act in ((bias, shc.SHC_ACT_RELU), (None, shc.SHC_ACT_NONE)):
        bd = None if b is None else up(b)
        out = torch.full((n + 3, Cout), float("nan"), dtype=TORCH[dtype], device=dev)
        direct = torch.full_like(out, float("nan"))
        shc.sparse_neighbor_conv_table(Sd, table, n, Wd, bd, out, act)
        shc.sparse_neighbor_conv(Sd, c.coords, c.inv, n, B, V, nd, Wd, bd, direct, act)
        got = down(out)
        assert np.all(np.isnan(got[n:])) and np.all(np.isnan(down(direct)[n:]))
        assert torch.equal(out[:n], direct[:n])
        ref = O.conv_at(S, coords, B, V, oob, W, rows, b, act=act == shc.SHC_ACT_RELU)
        scale = O.conv_at(S, coords, B, V, oob, W, rows, b, scale=True)
        assert_scaled_close(got[rows], ref, scale, dtype,
                            f"conv n={n} K={K} {Cin}->{Cout} act={act}", n_terms=K * Cin)


@pytest.mark.parametrize("what", ["tiny rows", "huge rows", "infinite rows", "NaN rows",
                                  "huge weights", "tiny weights"])
def test_conv_walk_value_range(dev, what):
    """fp32 products formed from bf16 terms, on values at the ends of fp32's
    range: rows whose sums leave the form's own range go to the fp32 matrix
    cores, every row stays within the fp32 bound, and infinities and NaN come
    out as in 64 bits."""
    B, V, n, K, Cin, Cout = 40, 655, 17001, 9, 128, 128
    rng = np.random.default_rng(len(what))
    nbr = rng.integers(0, V, size=(V, K)).astype(np.int32)
    nbr[:, 0] = np.arange(V)
    m = np.zeros(B * V, dtype=np.uint8)
    m[rng.permutation(B * V)[:n]] = 1
    m = m.reshape(B, V)
    c = Compaction(m)
    assert c.run() == n
    S = rng.standard_normal((n, Cin)).astype(np.float32)
    W = (rng.standard_normal((K, Cin, Cout)) / np.sqrt(K * Cin)).astype(np.float32)
    odd = rng.choice(n, 40, replace=False)
    if what == "tiny rows":
        S *= np.float32(1e-33)
    elif what == "huge rows":
        S[odd] *= np.float32(1e36)
    elif what == "infinite rows":
        S[odd, 3] = np.inf
        S[odd[:10], 5] = -np.inf
    elif what == "NaN rows":
        S[odd, 7] = np.nan
    elif what == "huge weights":
        W[2] *= np.float32(1e30)
    else:
        W *= np.float32(1e-34)
    coords, _, _, _ = O.compact(m)
    rows = np.unique(np.concatenate([odd, np.arange(300), rng.choice(n, 500, replace=False)]))
    nd = up(nbr)
    table = torch.empty(K * n, dtype=torch.int32, device=dev)
    shc.build_neighbor_table(c.coords, c.inv, n, B, V, nd, table)
    out = torch.full((n, Cout), float("nan"), dtype=torch.float32, device=dev)
    shc.sparse_neighbor_conv_table(up(S), table, n, up(W), None, out, shc.SHC_ACT_NONE)
    got = down(out)[rows]
    with np.errstate(all="ignore"):
        ref = O.conv_at(S.astype(np.float64), coords, B, V, nbr, W.astype(np.float64), rows, None)
        scale = O.conv_at(S.astype(np.float64), coords, B, V, nbr, W.astype(np.float64), rows,
                          None, scale=True)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], ref[inf])
    ok = np.isfinite(ref)
    # 1e-5 of the abs-sum scale, and the spacing of fp32's smallest numbers for
    # each of the K Cin products and sums below its normal range
    assert np.all(np.abs(got[ok] - ref[ok]) <= 1e-5 * scale[ok] + 2 * K * Cin * 2.0 ** -149)


def split_problem(dev, n, K, Cin, Cout, seed, keep=1.0):
    """Bodies, lists, table and values of a shape whose fp32 products are split
    (on the GPU); features are post-activation values, `keep` of them nonzero."""
    g = torch.Generator(device=dev).manual_seed(seed)
    B, V = 64, (n + 31) // 32
    nbr = torch.randint(0, V, (V, K), generator=g, device=dev, dtype=torch.int32)
    nbr[:, 0] = torch.arange(V, device=dev)
    m = np.zeros(B * V, dtype=np.uint8)
    m[np.random.default_rng(seed).permutation(B * V)[:n]] = 1
    c = Compaction(m.reshape(B, V))
    assert c.run() == n
    S = torch.randn((n, Cin), generator=g, device=dev).abs()
    S *= torch.rand((n, Cin), generator=g, device=dev) < keep
    W = torch.randn((K, Cin, Cout), generator=g, device=dev) / (K * Cin) ** 0.5
    table = torch.empty(K * n, dtype=torch.int32, device=dev)
    shc.build_neighbor_table(c.coords, c.inv, n, B, V, nbr, table)

    def conv(S, W, bias=None, coords=False):
        out = torch.full((n, Cout), float("nan"), device=dev)
        if coords:
            shc.sparse_neighbor_conv(S, c.coords, c.inv, n, B, V, nbr, W, bias, out,
                                     shc.SHC_ACT_NONE)
        else:
            shc.sparse_neighbor_conv_table(S, table, n, W, bias, out, shc.SHC_ACT_NONE)
        return out

    return S, W, table.view(K, n), conv


def dense_products(S, W, table, bias=None):
    """The conv and its sum of absolute products in 64 bits."""
    ref = torch.zeros((S.shape[0], W.shape[2]), dtype=torch.float64, device=S.device)
    if bias is not None:
        ref += bias.double()
    scale = ref.abs()
    for j in range(W.shape[0]):
        r = table[j].long()
        x = S.double()[r.clamp(min=0)] * (r >= 0)[:, None]
        ref += x @ W[j].double()
        scale += x.abs() @ W[j].double().abs()
    return ref, scale


def bits(t):
    """int32 view with one NaN pattern."""
    return torch.where(torch.isnan(t), torch.full_like(t, float("nan")), t).view(torch.int32)


@pytest.mark.parametrize("n", [17001, 33500])  # 256- and 128-row workgroups
@pytest.mark.parametrize("what", ["infinite", "huge", "tiny"])
def test_conv_walk_split_rows_apart(dev, n, what):
    """Infinite, huge (outside the split's range) and tiny values change the sums
    of the rows that use them and of no other: rows that do not have the same bits as without them,
    in every launch and from coordinates, whichever rows share a wavefront."""
    S, W, table, conv = split_problem(dev, n, 9, 128, 128, n)
    plain = conv(S, W)
    odd = torch.zeros(n, dtype=torch.bool, device=dev)
    odd[torch.from_numpy(np.random.default_rng(n).choice(n, 40, replace=False)).to(dev)] = True
    T = S.clone()
    if what == "infinite":
        T[odd, 3] = float("inf")
    elif what == "huge":
        T[odd] *= 2.0 ** 100
    else:
        T[odd] *= 2.0 ** -110
    uses = ((table >= 0) & odd[table.clamp(min=0).long()]).any(0)
    assert 0 < int(uses.sum()) < n // 2
    got = conv(T, W)
    assert torch.equal(bits(got)[~uses], bits(plain)[~uses])
    for coords in (False, True, False, True):
        assert torch.equal(bits(conv(T, W, coords=coords)), bits(got))


@pytest.mark.parametrize("what", ["weight column", "input channel", "products",
                                  "subnormal inputs", "subnormal weights"])
def test_conv_walk_split_mixed_magnitudes(dev, what):
    """Tiny values beside ordinary ones keep their precision: a weight column of
    2^-120 among ordinary columns, an input channel of 2^-120 whose neighbours
    meet zero weights, products near the smallest normal number, and inputs or
    weights below it.  Against
    64 bits relative to each output's sum of absolute products: fp32 sums of
    K Cin terms err by less than K Cin 2^-24 of it, and by 2^-149 an operation
    below fp32's normal range."""
    n, K, Cin, Cout = 17001, 9, 128, 128
    S, W, table, conv = split_problem(dev, n, K, Cin, Cout, 5)
    if what == "weight column":
        W[:, :, 17] *= 2.0 ** -120
    elif what == "input channel":
        S[:, 5] *= 2.0 ** -120
        W[:, :5] = 0
        W[:, 6:] = 0
        W[:, 5] *= 2.0 ** 20
    elif what == "products":
        S *= 2.0 ** -60
        W *= 2.0 ** -62
    else:
        small, large = (S, W) if what == "subnormal inputs" else (W, S)
        small *= 2.0 ** -132
        large *= 2.0 ** 30
        assert bool(((small != 0) & (small.abs() < 2.0 ** -126)).any())
    ref, scale = dense_products(S, W, table)
    err = (conv(S, W).double() - ref).abs()
    # a random walk of the roundings: 4e-7 seen, 1e-6 of the scale allowed (a
    # value kept to 16 bits errs by 2^-17 = 7.6e-6)
    assert bool((err <= 1e-6 * scale + 2 * K * Cin * 2.0 ** -149).all()), \
        float((err / scale.clamp(min=1e-300)).max())


@pytest.mark.parametrize("n,K,Cin,Cout", [(17001, 9, 128, 128), (33500, 9, 128, 128),
                                          (40001, 3, 144, 80), (23000, 20, 48, 80)])
@pytest.mark.parametrize("keep", [1.0, 0.5, 0.1, 0.03, 0.004])
@pytest.mark.parametrize("with_bias", [False, True])
def test_conv_walk_split_error(dev, n, K, Cin, Cout, keep, with_bias):
    """The split's 2-norm error against 64 bits is no larger than the fp32
    matrix cores' on the same values, from dense features to a few nonzero ones
    a row.  Sums times 2^100 are outside the split's range and take the fp32
    path: the same sums, scaled exactly."""
    S, W, table, conv = split_problem(dev, n, K, Cin, Cout, n + K, keep)
    bias = torch.randn(Cout, device=dev, generator=torch.Generator(dev).manual_seed(1)) \
        if with_bias else None
    ref, _ = dense_products(S, W, table, bias)
    big = None if bias is None else bias * 2.0 ** 100
    split = (conv(S, W, bias).double() - ref).norm() / ref.norm()
    chain = (conv(S, W * 2.0 ** 100, big).double() * 2.0 ** -100 - ref).norm() / ref.norm()
    print(f"n={n} K={K} {Cin}->{Cout} keep={keep} bias={with_bias}: split {split:.3e} fp32 {chain:.3e}")
    # equal roundings where a row has few products: 1% for their chance
    assert split <= 1.01 * chain, (float(split), float(chain))
