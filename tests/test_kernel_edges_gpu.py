"""Edges of the prefill kernels' tiles, units and list lengths, against the oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import superlinear as orc
from paper_2601_18401_amd import binding as B
from tests.test_parity_gpu import DEV, check_attention, f64, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Lq,k", [(1, 3), (63, 9), (64, 4), (65, 8), (129, 5), (1025, 12), (193, 32)])
def test_bucketing_units_and_list_lengths(Lq, k):
    """Row counts around the 64-row units of the bucketing passes, list lengths that are no whole 16-byte
    pieces, and rows that all list the same spans (one counter for the whole unit)."""
    S, L = 64, 64 * 40 + 17
    q0 = L - Lq
    Q, K, V = make(400 + Lq, 8, 2, L, 128, torch.bfloat16, Lq=Lq)
    idx = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0)
    same = idx.clone()
    same[:, :, :] = idx[:, :1, :]      # spans of the first row: candidates of every later one
    for sel in (idx, same):
        O, LSE = B.sl_span_attention_prefill(Q, K, V, sel, S, q_pos0=q0)
        torch.cuda.synchronize()
        rows = [(h, r) for h in range(8) for r in sorted({0, 1, Lq // 2, Lq - 1, *range(0, Lq, 67)}) if r < Lq]
        check_attention(O, LSE, Q, K, V, sel, S, q0, 0.0, rows)


@pytest.mark.parametrize("L,w,b,f", [(130, 1, 2, 0), (700, 63, 1, 1), (700, 64, 4, 2), (701, 65, 0, 0), (1500, 1088, 3, 2)])
def test_masked_kv_tiles_of_the_papers_geometry(L, w, b, f):
    """Ranges that start and end around the 64-token kv tiles, rows whose whole wavefront passes a tile over:
    the matrix-core form against the row-stationary form.  Weights, partials and outputs are rounded to bf16
    (2^-9 each) against outputs alone: 3 * 2^-9 * max|V| (about 4.5) plus 2^-9 * max|O|."""
    Q, K, V = make(500 + L, 8, 2, L, 128, torch.bfloat16, scale=0.5)
    an, sc = B.sl_anchor_search_prefill(Q, K, 3, w, want_scores=True)
    O = B.sl_anchor_attention_prefill(Q, K, V, an, sc, w, b, f)
    R = B.sl_anchor_attention_prefill(Q, K, V, an, sc, w, b, f, row_stationary=True)
    torch.cuda.synchronize()
    assert float((O.float() - R.float()).abs().max()) <= 3e-2
    assert float((O.float() - R.float()).abs().mean()) <= 2e-3


@pytest.mark.parametrize("Lq,S,A", [(64, 64, 64), (127, 192, 192), (129, 192, 64), (257, 320, 320)])
def test_masked_kv_tiles_on_the_grid(Lq, S, A):
    """Causal windows and clipped overlapping spans whose ends meet the kv tiles and the 128-row tiles."""
    L = 320 * 6 + 33
    q0 = L - Lq
    Q, K, V = make(600 + Lq, 4, 2, L, 128, torch.bfloat16, Lq=Lq)
    idx = B.sl_span_search_prefill(Q, K, None, A, 5, q_pos0=q0)
    O, LSE = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0, span_stride=A)
    torch.cuda.synchronize()
    check_attention(O, LSE, Q, K, V, idx, S, q0, 0.0, [(h, r) for h in range(4) for r in range(0, Lq, 3)], stride=A)
