"""Branches of the launch rules (how many rows, keys or columns a workgroup takes, by the size of the problem): each at the
sizes where it can go wrong, against the oracle.  Tolerances: REL_TOL for bf16 outputs; 1e-4 for 32-bit sums of
exponentials, whose argument, below 32 in magnitude, is rounded to 2^-19 at most twice (2 * 2^-19 * ln 2 = 2.6e-6 of a
weight) before a sum of up to 192 positive terms (192 * 2^-24 = 1.1e-5)."""
import math

import numpy as np
import pytest
import torch

import synth_inputs as si
import parity as recipes
from parity import REL_TOL, rel_err

pytestmark = pytest.mark.gpu

DEV = "cuda"
SUM_TOL = 1e-4


@pytest.fixture(scope="module")
def cm():
    import paper_2506_03275_amd as cm
    cm.load()
    return cm


def _u8(nbytes):
    return torch.empty(max(int(nbytes), 16), dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("N,E,c", [(1, 128, 192), (64, 64, 128), (130, 128, 192), (511, 64, 192), (513, 128, 128),
                                   (1100, 128, 192), (2113, 64, 128), (2113, 128, 192)])   # 1, 1, 1, 2, 2, 4, 8, 8 pieces
def test_column_sums_in_pieces_of_the_keys(cm, oracle, N, E, c):
    """The column-sum pass cuts a chunk's keys into 1 to 8 runs of 64-key tiles, the last tile ragged or not."""
    (q, k, _), _, _ = si.attn_steps(1, 1, N, E, 21, DEV)
    scale, NB, ld = 1 / math.sqrt(E), -(-N // c), -(-N // 4) * 4 + 4
    m_ref, l_ref = oracle.attn_row_stats(si.np_f32(q), si.np_f32(k), scale)
    m = torch.from_numpy(m_ref.astype(np.float32) - 0.25).to(DEV)
    l = torch.from_numpy(l_ref.astype(np.float32) * 1.5).to(DEV)
    D = torch.full((1, 1, NB, ld), -1.0, dtype=torch.float32, device=DEV)
    cm.attn_colsum_stale(q, k, m, l, D, c, scale)
    ref = oracle.attn_colsum_stale(si.np_f32(q), si.np_f32(k), m.cpu().numpy().astype(np.float64),
                                   l.cpu().numpy().astype(np.float64), c, scale)
    got = D.cpu().numpy()
    assert rel_err(got[..., :N].astype(np.float64), ref) <= SUM_TOL
    assert (got[..., N:] == -1.0).all()
