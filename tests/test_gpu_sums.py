"""The errors of the 32-bit sums: not only that they stay below a tolerance of the whole path, but that they are as small as
the arithmetic allows."""
import ctypes
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


@pytest.mark.parametrize("chunks,D,F,plan", [
    (1, 128, 64, (0, 0)), (8, 256, 1024, (0, 0)), (8, 1792, 1024, (0, 0)),         # the kernel for few chunks
    (14, 2048, 8704, (0, 0)), (24, 3072, 12288, (0, 0)),
    (300, 384, 2048, (1, 2)),                                 # one piece, two sums
    (1, 4864, 64, (16, 2)), (60, 4096, 1088, (16, 2)), (24, 3072, 10240, (3, 2)),   # 16 and 3 pieces, two sums each
    (48, 5120, 12224, (5, 1)), (129, 512, 8576, (3, 1)),      # five pieces and three, one sum each
    (40, 4096, 10240, (4, 2)),                                # four pieces, two sums each: fewer would be too long
    (258, 1024, 6912, (2, 2)), (129, 1024, 16640, (1, 2)),    # two pieces and one, two sums each
    (602, 1024, 12288, (1, 1)),                               # one piece, one sum
])
def test_neuron_scores_add_no_longer_sums_than_the_workspace_has_pieces_for(cm, chunks, D, F, plan):
    """Chunk means that two bf16 numbers hold exactly, so that what is left is the error of the GEMM's 32-bit sums.  One rounding
    of the result is 2^-23 * sqrt(0.52 / 12) in the mean square (0.52: of the squared mantissas).  Eight products are added
    with one rounding, so D / 8 additions in h chains of the high parts leave D / 16 / h of its variance; merging h chains of
    high and as many of low parts leaves 1.5 h.  h is half of the pieces that the workspace is sized for."""
    c = 128
    form = (ctypes.c_int32 * 5)()
    cm.load().chipmunk_internal_mlp_form(1, chunks * c, D, F, c, 1, chunks * c, form)
    assert tuple(form[3:]) == plan
    g = si.generator(32, DEV)
    pair = (1 + torch.randint(0, 128, (2, chunks, D), generator=g, device=DEV) / 128)
    pair = pair * (1 - 2 * torch.randint(0, 2, (chunks, D), generator=g, device=DEV))
    x = pair.permute(1, 0, 2)[:, None].expand(chunks, c // 2, 2, D).reshape(1, chunks * c, D).to(torch.bfloat16)
    w1 = si.randn_bf16((F, D), g, 1 / math.sqrt(D))
    ws = torch.empty(max(cm.mlp_tile_mean_workspace_bytes(1, chunks * c, D, F, c), 16), dtype=torch.uint8, device=DEV)
    T = torch.empty((1, chunks, F), dtype=torch.float32, device=DEV)
    cm.mlp_tile_mean_preact(x, w1, T, c, ws)
    ref = pair.to(F64).mean(0) @ w1.to(F64).t().contiguous()
    h = min(max((ws.numel() - chunks * D * 4) // (chunks * F * 4) // 2, 1), D // 64)
    bound = 2.0 ** -23 * math.sqrt(0.52 / 12 * (D / 16 / h + 1.5 * h))
    # a rounding is counted at the mean square of its sum; a few sums of small problems scatter around that
    assert _rms_err(T[0], ref) <= bound * (1 + 2 / math.sqrt(chunks * F))
    again = torch.empty_like(T)
    cm.mlp_tile_mean_preact_static(x, w1, again, c)
    assert _rms_err(again[0], ref) <= bound * (1 + 2 / math.sqrt(chunks * F)) or chunks * (D + F) * 4 > 1 << 25
