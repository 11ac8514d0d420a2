"""The sparse neighbour conv from a table on the shapes its slot-major kernel
serves (64 input channels within one round of row groups, and dense masks
with about a thousand rows or more per CU): Eqs. 4-5 against the oracle on
sampled rows, with and without bias and ReLU, rows past N' untouched.  The
bit-for-bit agreement with the weight-stationary kernel is checked where both
run on the same inputs (the planned conv of the plan tests at 64 channels).
Every input is seeded and synthetic.
"""
import numpy as np
import pytest
import torch

from oracle import shc_oracle as O
from paper_2608_09388_amd import binding as shc
from paper_2608_09388_amd import synth
from tests.gpu_util import Compaction, assert_scaled_close, down, require_gpu, up

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def rand_nbr(V, K, rng, p_missing=0.1):
    nbr = rng.integers(0, V, size=(V, K)).astype(np.int32)
    nbr[rng.random((V, K)) < p_missing] = -1
    nbr[:, 0] = np.arange(V)
    return nbr


@pytest.mark.parametrize("B,V,K,Cin,Cout,p,mesh", [
    (64, 655, 9, 64, 64, 0.1, False),      # the encoder's 64 -> 64 layer
    (64, 655, 9, 64, 128, 0.1, False),     # and its 64 -> 128 layer
    (3, 700, 5, 64, 64, 0.4, False),       # K other than nine (a loop over the slots)
    (2, 300, 1, 64, 128, 0.6, False),      # one slot
    (4, 400, 32, 64, 64, 0.3, False),      # 32 slots
    (1, 40, 9, 64, 64, 0.5, False),        # one partial row group
    (128, 10475, 9, 128, 128, 0.2, True),  # the density-sweep batch at 20%
    (256, 10475, 9, 64, 64, 0.18, True),   # the full-mesh batch, cap-like density
])
def test_conv_sm_shapes_against_oracle(dev, B, V, K, Cin, Cout, p, mesh):
    rng = np.random.default_rng(B + V + 7 * K + Cin + Cout)
    if mesh:
        _, nbr = synth.mesh("ellipsoid", V, K, 4)
        nbr = np.ascontiguousarray(nbr, dtype=np.int32)
    else:
        nbr = rand_nbr(V, K, rng)
    m = (rng.random((B, V)) < p).astype(np.uint8)
    c = Compaction(m)
    n = c.run()
    table = torch.full((max(K * n, 1),), -7, dtype=torch.int32, device=dev)
    shc.build_neighbor_table(c.coords, c.inv, n, B, V, up(nbr), table)
    S = synth.as_dtype(rng.standard_normal((n, Cin)).astype(np.float32), "bf16")[1]
    W = synth.as_dtype((rng.standard_normal((K, Cin, Cout)) / np.sqrt(K * Cin))
                       .astype(np.float32), "bf16")[1]
    bias = rng.standard_normal(Cout).astype(np.float32)
    coords, _, _, n_ref = O.compact(m)
    assert n_ref == n
    rows = np.unique(np.concatenate([np.arange(min(n, 200)), np.arange(max(0, n - 200), n),
                                     rng.choice(n, size=min(n, 400), replace=False)]))
    Sd, Wd = up(S, "bf16"), up(W, "bf16")
    for b, act in ((bias, shc.SHC_ACT_RELU), (None, shc.SHC_ACT_NONE)):
        out = torch.full((n + 3, Cout), float("nan"), dtype=torch.bfloat16, device=dev)
        shc.sparse_neighbor_conv_table(Sd, table, n, Wd, None if b is None else up(b), out, act)
        got = down(out)
        assert np.all(np.isnan(got[n:]))
        ref = O.conv_at(S, coords, B, V, nbr, W, rows, b, act=act == shc.SHC_ACT_RELU)
        scale = O.conv_at(S, coords, B, V, nbr, W, rows, b, scale=True)
        assert_scaled_close(got[rows], ref, scale, "bf16",
                            f"conv K={K} {Cin}->{Cout} p={p} act={act}", n_terms=K * Cin)
    torch.cuda.synchronize()


# 128- and 192-row workgroups, two to a CU, their output staged where the weights
# were: eight wavefronts and four, a last group that is nearly empty, one and two
# slots (the staging tiles then reach past the weights), an odd and an even
# slot count of the loop, and the 320-row form where two do not fit; then either
# side of the lines to the tiled kernel (few slots, short and wide reductions,
# wide outputs); rows past N' untouched.
@pytest.mark.parametrize("n,K,Cin,Cout", [
    (129, 1, 64, 128), (2 * 128 + 1, 2, 64, 64), (65536, 5, 64, 64), (65537, 9, 64, 64),
    (65537, 6, 64, 64), (40001, 12, 128, 64), (32769, 11, 128, 128), (32900, 14, 128, 128),
    (256000, 9, 128, 64), (256003, 15, 128, 128),
    (192 * 1334 + 1, 9, 128, 128), (256000 + 191, 1, 128, 128), (33001, 10, 128, 128),
    (32768, 5, 48, 80), (32769, 5, 48, 80), (16384, 5, 16, 256), (16385, 5, 16, 256),
    (32769, 12, 96, 256),
])
def test_conv_sm_workgroups_against_dense_products(dev, n, K, Cin, Cout):
    g = torch.Generator(device=dev).manual_seed(n + K)
    table = torch.randint(0, n, (K, n), generator=g, device=dev, dtype=torch.int32)
    table[torch.rand((K, n), generator=g, device=dev) < 0.6] = -1
    S = torch.randn((n, Cin), generator=g, device=dev).to(torch.bfloat16)
    W = (torch.randn((K, Cin, Cout), generator=g, device=dev) / (K * Cin) ** 0.5).to(torch.bfloat16)
    bias = torch.randn(Cout, generator=g, device=dev)
    out = torch.full((n + 1, Cout), float("nan"), dtype=torch.bfloat16, device=dev)
    shc.sparse_neighbor_conv_table(S, table, n, W, bias, out, shc.SHC_ACT_RELU)
    rows = torch.cat([torch.arange(min(n, 300)), torch.arange(max(0, n - 300), n),
                      torch.arange(0, n, max(1, n // 500))]).to(dev)
    ref = bias.double().expand(len(rows), Cout).clone()
    scale = ref.abs()
    for j in range(K):
        src = table[j][rows].long()
        x = torch.where((src >= 0)[:, None], S[src.clamp(min=0)], torch.zeros_like(S[:1])).double()
        ref += x @ W[j].double()
        scale += x.abs() @ W[j].double().abs()
    assert torch.isnan(out[n:]).all()
    assert_scaled_close(out[rows].float().cpu().numpy(), ref.clamp(min=0).cpu().numpy(),
                        scale.cpu().numpy(), "bf16", f"conv n={n} K={K} {Cin}->{Cout}",
                        n_terms=K * Cin)
