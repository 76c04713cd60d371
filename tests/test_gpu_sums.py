"""The errors of the 32-bit sums: not only that they stay below a tolerance of the whole path, but that they are as small as
the arithmetic allows."""
import math

import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu

DEV = "cuda"
F64 = torch.float64


@pytest.fixture(scope="module")
def cm():
    import paper_2506_03275_amd as cm
    cm.load()
    return cm


def _rms_err(got, ref):
    return float((got.to(F64) - ref).norm() / ref.norm())


@pytest.mark.parametrize("N,E,c", [(1538, 64, 128), (1154, 64, 192), (1538, 128, 128), (4608, 128, 192)])
def test_column_sums_of_given_normalisers(cm, N, E, c):
    """A weight exp(s - m) / l has one rounding of its argument (below 16 in magnitude: at most 2^-21, 2^-21 / sqrt(3) in the
    mean square, times ln 2: 1.9e-7 of the weight), as much from m in units of log2, and 2^-23 from the exponential and from
    1 / l: 2.9e-7 together, independent from row to row.  A column adds 128 or 192 weights that are spread like exp of a
    normal score, which count as at least 45 equal ones: 4.3e-8, and the sum of the weights itself has 4e-8.  1.2e-7 is twice
    what that makes.  A normaliser that enters the argument as a logarithm, at twice the magnitude, does not meet it
    (1.9e-7 and more)."""
    H = 3
    g = si.generator(31, DEV)
    q, k = (si.randn_bf16((1, H, N, E), g) for _ in range(2))
    scale, NB = 1 / math.sqrt(E), -(-N // c)
    scores = torch.matmul(q[0].to(F64), k[0].to(F64).transpose(1, 2).contiguous()) * scale
    m = (scores.amax(-1) - 0.25).float()
    l = (torch.exp(scores - m[..., None].to(F64)).sum(-1) * 1.5).float()
    D = torch.zeros((1, H, NB, -(-N // 4) * 4), dtype=torch.float32, device=DEV)
    cm.attn_colsum_stale(q, k, m[None].contiguous(), l[None].contiguous(), D, c, scale)
    weights = torch.exp(scores - m[..., None].to(F64)) / l[..., None].to(F64)
    ref = torch.stack([weights[:, u * c:(u + 1) * c].sum(1) for u in range(NB)], 1)
    assert _rms_err(D[0, :, :, :N], ref) <= 1.2e-7
