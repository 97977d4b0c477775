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
