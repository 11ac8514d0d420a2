"""Kernels whose workgroup size or launch count follows the problem's size, at
the sizes where that changes: the compaction of masks at the limit below which
it takes one launch (lists, table and slot pairs), group norm and max-pool over
many short bodies (their smaller workgroups, bodies of more rows than stay in
registers), and the transposed table at the edges of its 64-row blocks.
Against the oracle or its definition written out; every input is seeded.
"""
import numpy as np
import pytest
import torch

from oracle import shc_oracle as O
from paper_2608_09388_amd import binding as shc
from paper_2608_09388_amd import synth
from tests.gpu_util import (TORCH, assert_gn_close, down, gn_floor, require_gpu, up)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


# B above the CU count: workgroups of 256, 512 or 1024 threads by the mean row
# count; body 3 is full (more rows than stay in registers), 1 and B - 1 empty
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,V,C,G,p", [(300, 400, 32, 8, 0.12), (600, 655, 256, 32, 0.1),
                                       (280, 300, 96, 4, 0.5), (270, 700, 256, 1, 0.4)])
def test_short_bodies_norm_and_pool(dev, dtype, B, V, C, G, p):
    rng = np.random.default_rng(B + V + C)
    m = (rng.random((B, V)) < p).astype(np.uint8)
    m[[1, B - 1]] = 0
    m[3] = 1
    m[4] = 0
    m[4, 7] = 1
    coords, inv, rp, n = O.compact(m)
    S = (rng.standard_normal((n, C)) * 2.0 + rng.standard_normal(C) * 3.0).astype(np.float32)
    S = synth.as_dtype(S, dtype)[1]
    Sd = up(S, dtype)
    out = torch.full((n + 3, C), float("nan"), dtype=TORCH[dtype], device=dev)
    shc.segment_group_norm(Sd, up(rp), n, B, G, out)
    got = down(out)
    assert np.all(np.isnan(got[n:]))
    assert_gn_close(got[:n], O.group_norm(S.astype(np.float64), rp, G), dtype,
                    gn_floor(S, rp, G), f"group norm B={B} C={C} G={G}")
    P = torch.full((B, C), float("nan"), dtype=TORCH[dtype], device=dev)
    shc.segment_maxpool(Sd, up(rp), n, B, P, -2.0)
    assert np.array_equal(down(P), O.segment_max(S.astype(np.float64), rp, -2.0))
