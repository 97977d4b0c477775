"""Edges of the prefill kernels' tiles, units and list lengths, against the oracle."""
import ctypes
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


FINE = [
    # Hq Hkv L     D    S    A    k  form     q_pos0 Lq
    (8, 2, 6000, 128, 77, 77, 8, "joint", 0, 6000),       # odd span length
    (8, 2, 6000, 64, 64, 64, 5, "joint", 0, 6000),        # D = 64
    (4, 4, 9001, 64, 95, 95, 4, "gated", 0, 9001),
    (8, 2, 7000, 128, 130, 130, 9, "joint", 1000, 6000),  # more slots than the short merge takes
    (8, 1, 5000, 128, 150, 75, 8, "joint", 0, 5000),      # overlapping spans, odd spacing
    (8, 1, 5000, 128, 150, 50, 17, "gated", 0, 5000),
    (16, 2, 3000, 128, 33, 33, 8, "joint", 17, 2900),     # barely longer than half a kv tile
]


@pytest.mark.parametrize("S,k,q_pos0,Lq", [(64, 7, 0, 1300), (64, 9, 300, 700), (128, 16, 1900, 300), (64, 17, 900, 400),
                                          (64, 25, 0, 2000), (64, 32, 1900, 300)])
def test_gated_merge_of_rows_with_and_without_a_full_list(S, k, q_pos0, Lq):
    """Rows on both sides of position k * S, from which on there are candidates for all slots, lists of one and of
    several batches of partials, and empty slots in the middle of lists."""
    from tests.test_parity_gpu import check_combined
    L = q_pos0 + Lq
    Q, K, V = make(1400 + k, 4, 2, L, 128, torch.bfloat16, Lq=Lq, scale=0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q_pos0, want_scores=True)
    sc = torch.where(torch.isfinite(sc), sc, 0.0)
    holes = idx.clone()
    holes[:, ::2, ::3] = -1
    holes[:, 1::4, 1] = 4000      # no candidate of any row
    rows = [(h, r) for h in range(4) for r in sorted({0, 1, Lq - 1, *range(0, Lq, 29),
                                                      *(x for x in range(k * S - q_pos0 - 3, k * S - q_pos0 + 3) if 0 <= x < Lq)})]
    for sel in (idx, holes):
        O = B.sl_span_attention_combined_prefill(Q, K, V, sel, sc, S, q_pos0=q_pos0)
        torch.cuda.synchronize()
        check_combined(O, Q, K, V, sel, sc, S, q_pos0, 0.0, rows)


def row_form(Q, K, V, idx, sc, S, q_pos0=0, span_stride=0):
    """The row-stationary kernels, which a call without a workspace runs: (O, LSE), or O where sc is given."""
    p = B.make_params(Q, K, S, idx.shape[2], q_pos0, 0.0, span_stride)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    R, RL = torch.empty_like(Q), torch.empty(Q.shape[:2], dtype=torch.float32, device=DEV)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if sc is None:
        st = B.load().sl_span_attention_prefill(ctypes.byref(p), ptr(Q), ptr(K), ptr(V), ptr(idx), ptr(R), ptr(RL),
                                                None, 0, stream)
    else:
        st = B.load().sl_span_attention_combined_prefill(ctypes.byref(p), ptr(Q), ptr(K), ptr(V), ptr(idx), ptr(sc),
                                                         ptr(R), None, 0, stream)
    assert st == B.SL_OK
    return (R, RL) if sc is None else R


def takes_matrix_cores(Q, K, S, k, q_pos0=0, span_stride=0):
    return B.workspace_bytes(B.make_params(Q, K, S, k, q_pos0, 0.0, span_stride), B.OP_ATTENTION_PREFILL) > 0


@pytest.mark.parametrize("Hq,Hkv,L,D,S,A,k,form,q_pos0,Lq", FINE)
def test_any_span_length_on_the_matrix_cores(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq):
    """Span lengths that are no multiple of 64 and D = 64: the matrix-core form with split weights against the
    row-stationary kernels (a workspace of zero bytes selects them), which the oracle covers.  Both keep the
    weights and partial sums in fp32 and round the output to bf16 once: they differ by at most one bf16 step of
    it, 2^-7 relative.  Their sums run in different orders, so with finite inputs some roundings turn: an output
    equal to the last bit would be the recomputation by the row-stationary kernels, which an output that is not
    finite starts."""
    stride = 0 if A == S else A
    std = 1.0 if form == "joint" else 0.35
    Q, K, V = make(700 + L + S, Hq, Hkv, L, D, torch.bfloat16, Lq=Lq, scale=std)
    idx, sc = B.sl_span_search_prefill(Q, K, None, A, k, q_pos0=q_pos0, want_scores=True)
    assert takes_matrix_cores(Q, K, S, k, q_pos0, stride)
    if form == "joint":
        O, LSE = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q_pos0, span_stride=stride)
        R, RL = row_form(Q, K, V, idx, None, S, q_pos0, stride)
    else:
        O = B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, q_pos0=q_pos0, span_stride=stride)
        R = row_form(Q, K, V, idx, sc, S, q_pos0, stride)
    torch.cuda.synchronize()
    o, r = O.float(), R.float()
    assert float(((o - r).abs() - r.abs() * 2 ** -7).max()) <= 1e-4
    turned = float((o != r).float().mean())    # sums of some hundred fp32 terms: 2^-20 and less against steps of 2^-8
    assert 0.0 < turned <= 0.02, turned
    if form == "joint":
        assert float((LSE - RL).abs().max()) <= 1e-5


@pytest.mark.parametrize("Hq,Hkv,L,D,S,A,k,form,q_pos0,Lq", [
    (12, 2, 15272, 64, 1920, 960, 12, "gated", 15152, 120),
    (4, 1, 3000, 64, 1441, 1441, 4, "joint", 2700, 300),
    (8, 2, 6000, 64, 129, 129, 8, "joint", 5700, 300),
    (64, 8, 8000, 64, 100, 100, 8, "joint", 7700, 300),
    (32, 4, 9000, 64, 600, 600, 8, "gated", 6000, 3000),
    (8, 2, 8000, 64, 81, 81, 8, "joint", 3900, 4100),
])
def test_long_and_short_spans_at_64_dimensions(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq):
    """Few tiles and many, one stage a span and thirty, with remainders, on test_any_span_length_on_the_matrix_cores's terms."""
    test_any_span_length_on_the_matrix_cores(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq)


def local_heads(G):
    return min(G & -G, 8)


def long_stages(Hq, Hkv, L, A, k, Lq):
    """Whether the routed and the window kernel of any span length (D = 128) stage 64 tokens, and not 32, at a time: where as many
    workgroups as 256 compute units hold of that form take all tiles at once."""
    n, G, items = -(-L // A), Hq // Hkv, Hq * Lq * k
    routed = min(items, Hkv * n) + items / 128
    rows = 128 // local_heads(G)
    tiles = -(-Lq // rows)
    run = max(1, min(A // rows, -(-tiles // 8)))
    chunks = -(-tiles // run)
    most = max((chunks - x + 7) // 8 * run - (chunks * run - tiles if (chunks - 1) % 8 == x else 0) for x in range(8))
    return routed <= 512, 8 * Hkv * most * (G // local_heads(G)) <= 512


@pytest.mark.parametrize("Hq,Hkv,L,D,S,A,k,form,q_pos0,Lq,routed,window", [
    (8, 2, 5100, 128, 417, 417, 4, "joint", 4900, 200, True, True),
    (8, 2, 5100, 128, 450, 225, 4, "gated", 4900, 200, True, True),
    (72, 72, 3391, 128, 838, 838, 4, "joint", 3351, 40, True, False),      # many kv heads: the grid of the windows is padded
    (72, 72, 3391, 128, 838, 838, 4, "gated", 3351, 40, True, False),
    (32, 4, 9001, 128, 47, 47, 8, "joint", 8501, 500, False, True),
    (32, 4, 9001, 128, 141, 47, 8, "joint", 8501, 500, False, True),
    (16, 4, 17001, 128, 65, 65, 8, "gated", 0, 17001, False, False),
    (16, 4, 17001, 128, 97, 97, 8, "joint", 0, 17001, False, False),
])
def test_stages_of_both_lengths(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq, routed, window):
    """Each choice of a stage's length for spans and windows, with remainders, on test_any_span_length_on_the_matrix_cores's terms."""
    assert long_stages(Hq, Hkv, L, A, k, Lq) == (routed, window)
    test_any_span_length_on_the_matrix_cores(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq)


def token_major(x):
    """The same values with the heads of a token side by side and a gap behind them."""
    H, T, D = x.shape
    buf = torch.full((T, H + 1, D), float("nan"), dtype=x.dtype, device=x.device)
    buf[:, :H] = x.transpose(0, 1)
    return buf[:, :H].transpose(0, 1)


@pytest.mark.parametrize("D,S,form", [(64, 64, "joint"), (128, 77, "joint"), (128, 77, "gated")])
def test_any_span_length_with_strided_inputs(D, S, form):
    """Token-major queries and caches with gaps: the packed inputs' result to the bit."""
    Q, K, V = make(810 + D, 8, 2, 6000, D, torch.bfloat16, Lq=5000, scale=0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, 8, q_pos0=1000, want_scores=True)
    q, kk, v = token_major(Q), token_major(K), token_major(V)
    assert takes_matrix_cores(q, kk, S, 8, 1000) and takes_matrix_cores(Q, K, S, 8, 1000)
    if form == "joint":
        a, b = (B.sl_span_attention_prefill(*x, idx, S, q_pos0=1000) for x in ((Q, K, V), (q, kk, v)))
    else:
        a, b = ((B.sl_span_attention_combined_prefill(*x, idx, sc, S, q_pos0=1000),) for x in ((Q, K, V), (q, kk, v)))
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, b)) and bool(torch.isfinite(a[0].float()).all())


@pytest.mark.parametrize("D,k", [(64, 2), (128, 4)])
def test_anchor_search_on_the_matrix_cores_with_strided_inputs(D, k):
    """Token-major queries and keys with gaps: the packed inputs' result to the bit."""
    L, q0 = 30000, 28500
    Q, K, _ = make(1150 + D, 8, 2, L, D, torch.bfloat16, Lq=L - q0, scale=0.5)
    a, b = (B.sl_anchor_search_prefill(*x, k, 24, q_pos0=q0, want_scores=True) for x in ((Q, K), (token_major(Q), token_major(K))))
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("form", ["joint", "gated"])
def test_any_span_length_in_several_passes_over_the_kv_heads(form):
    """More partials than 4 GiB of scratch hold: three kv heads, then the fourth, in the same workspace."""
    Hq, Hkv, L, D, S, k = 32, 4, 30011, 128, 174, 8
    std = 1.0 if form == "joint" else 0.35
    Q, K, V = make(820, Hq, Hkv, L, D, torch.bfloat16, scale=std)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, want_scores=True)
    need = B.workspace_bytes(B.make_params(Q, K, S, k), B.OP_ATTENTION_PREFILL)
    assert 3 * Hq // Hkv * L * (k + 1) * D * 4 < need < Hq * L * (k + 1) * D * 4
    if form == "joint":
        O, LSE = B.sl_span_attention_prefill(Q, K, V, idx, S)
        R, RL = row_form(Q, K, V, idx, None, S)
        assert float((LSE - RL).abs().max()) <= 1e-5
    else:
        O, R = B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S), row_form(Q, K, V, idx, sc, S)
    torch.cuda.synchronize()
    o, r = O.float(), R.float()
    assert float(((o - r).abs() - r.abs() * 2 ** -7).max()) <= 1e-4
    for kv in range(Hkv):
        turned = float((o != r)[kv * Hq // Hkv:(kv + 1) * Hq // Hkv].float().mean())
        assert 0.0 < turned <= 0.02, (kv, turned)


@pytest.mark.parametrize("D", [64, 128])
def test_any_span_length_keeps_fp32_weights(D):
    """Rows whose softmax is three keys and whose values cancel: the output is what the weights' rounding leaves.
    Against fp64 the matrix-core form must not be further off than twice the row-stationary form, whose weights are
    fp32: what both share is the rounding of the logits (measured 0.6 and 1.3 times as far; with weights of 16 to 17
    bits 2.8 and 3.5 times)."""
    Hq, Hkv, L, S, k = 16, 8, 4000, 77, 8
    Q, K, V = make(803 + D, Hq, Hkv, L, D, torch.bfloat16, scale=1.0)
    idx = B.sl_span_search_prefill(Q, K, None, S, k)
    assert takes_matrix_cores(Q, K, S, k)
    tailored, gen = [], torch.Generator().manual_seed(D)
    for kv in range(Hkv):
        h, r = 2 * kv + kv % 2, L - 1 - 5 * kv
        ts = [int(idx[h, r, 0]) * S + x for x in (3, 20, 41)]
        q = Q[h, r].double().cpu()
        for t, x in zip(ts, (8.0, 7.9, 7.6)):    # logits
            K[kv, t] = (q * (x * math.sqrt(D) / float(q @ q))).to(torch.bfloat16).to(DEV)
        spans = [int(j) for j in idx[h, r] if j >= 0]
        toks = torch.tensor(sorted({t for j in spans for t in range(j * S, j * S + S)} | set(range(r // S * S, r + 1))))
        p = torch.softmax(K[kv].double().cpu()[toks] @ q / math.sqrt(D), 0)
        v = V[kv].double().cpu()[toks]
        at = [int((toks == t).nonzero()) for t in ts]
        rest = p @ v - sum(p[a] * v[a] for a in at)
        v1 = torch.where(torch.rand(D, generator=gen) < 0.5, 1.0, -1.0).double()
        v2 = (-(rest + p[at[0]] * v1) / p[at[1]]).to(torch.bfloat16).double()
        v3 = (-(rest + p[at[0]] * v1 + p[at[1]] * v2) / p[at[2]]).to(torch.bfloat16).double()
        for t, x in zip(ts, (v1, v2, v3)):
            V[kv, t] = x.to(torch.bfloat16).to(DEV)
        tailored.append((h, r, rest + p[at[0]] * v1 + p[at[1]] * v2 + p[at[2]] * v3))
    O = B.sl_span_attention_prefill(Q, K, V, idx, S)[0]
    R = row_form(Q, K, V, idx, None, S)[0]
    torch.cuda.synchronize()
    off = [math.sqrt(sum(float(((X[h, r].double().cpu() - o) ** 2).mean()) for h, r, o in tailored) / Hkv) for X in (O, R)]
    assert off[0] <= 2 * off[1], off


@pytest.mark.parametrize("Hq,Hkv,L,D,S,k", [(32, 4, 5000, 128, 142, 8), (32, 4, 3000, 128, 55, 8), (8, 8, 9000, 128, 838, 2), (32, 4, 5000, 64, 90, 8)])
def test_any_span_length_rounds_lse_to_the_last_place(Hq, Hkv, L, D, S, k):
    """lse with nine roundings of partials that average out, the logarithm of their sum and the last addition, 0.3 of a unit in
    the last place each: 0.4 to 0.45 units are seen.  Logarithms of whole sums of weights, which lie at 16 to 64, added half as much."""
    Q, K, V = make(800 + S, Hq, Hkv, L, D, torch.bfloat16)
    Lq = min(L, 3000)
    Q, q0 = Q[:, -Lq:].contiguous(), L - Lq
    idx = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0)
    assert takes_matrix_cores(Q, K, S, k, q0)
    _, LSE = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0)
    torch.cuda.synchronize()
    rows = torch.arange(0, Lq, max(1, Lq // 300), device=DEV)
    pos, kv = q0 + rows, torch.arange(Hq, device=DEV)[:, None] // (Hq // Hkv)
    q, spans = Q[:, rows].double() / math.sqrt(D), idx[:, rows].long()
    parts = []
    for s in range(k + 1):
        start = spans[:, :, s] * S if s < k else (pos // S * S).expand(Hq, -1)
        at = start[:, :, None] + torch.arange(S, device=DEV)
        z = torch.stack([(K[kv[h], at[h].clamp(0, L - 1)].double() @ q[h, :, :, None])[..., 0] for h in range(Hq)])
        parts.append(z.masked_fill((at < 0) | (at > pos[None, :, None]), -math.inf).logsumexp(dim=2))
    want = torch.stack(parts).logsumexp(dim=0)
    units = (LSE[:, rows].double() - want) / torch.exp2(want.abs().log2().floor() - 23)
    assert float(units.pow(2).mean().sqrt()) <= 0.5


@pytest.mark.parametrize("form", ["joint", "gated"])
def test_optional_scratch_is_the_calls_own_and_can_be_missing(form, monkeypatch):
    """A call that can run without scratch leaves the binding's shared workspace alone, and where there is no room
    for the scratch it runs row by row."""
    Q, K, V = make(806, 8, 2, 6000, 64, torch.bfloat16, scale=0.35)
    S, k = 77, 8
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, want_scores=True)
    assert takes_matrix_cores(Q, K, S, k)

    def call(ws=None):
        return B.sl_span_attention_prefill(Q, K, V, idx, S, ws=ws)[0] if form == "joint" else \
            B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, ws=ws)
    R = row_form(Q, K, V, idx, None if form == "joint" else sc, S)
    R = R[0] if form == "joint" else R
    shared = B._ws(None)
    before = shared.buf
    monkeypatch.setattr(shared, "buf", None)
    O = call()
    assert shared.buf is None
    monkeypatch.setattr(shared, "buf", before)
    own = B.Workspace()
    O2 = call(own)
    assert own.buf is not None

    def no_room(self, nbytes):
        raise torch.cuda.OutOfMemoryError("no room")
    monkeypatch.setattr(B.Workspace, "get", no_room)
    N, N2 = call(), call(own)
    torch.cuda.synchronize()
    assert torch.equal(O, O2) and not torch.equal(O, R)
    assert torch.equal(N, R) and torch.equal(N2, R)


def test_armed_events_hold_the_routed_kernel_of_any_span_length():
    """The routed kernel is more than half of this call; the conditional recomputation behind it, which ends at
    once, is some microseconds."""
    Q, K, V = make(800, 32, 4, 12000, 128, torch.bfloat16)
    idx = B.sl_span_search_prefill(Q, K, None, 110, 8)
    assert takes_matrix_cores(Q, K, 110, 8)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()                      # creates the handles
    for _ in range(3):
        ev[0].record()
        B.sl_span_attention_prefill(Q, K, V, idx, 110, prof=(ev[1].cuda_event, ev[2].cuda_event))
        ev[3].record()
        torch.cuda.synchronize()
    whole, kernel = ev[0].elapsed_time(ev[3]), ev[1].elapsed_time(ev[2])
    assert 0.3 * whole < kernel < whole, (kernel, whole)


@pytest.mark.parametrize("form", ["joint", "gated"])
@pytest.mark.parametrize("span", [12, 40])     # a span that lies in no row's window; one that does
@pytest.mark.parametrize("which,bad", [("V", float("nan")), ("V", float("inf")), ("K", float("nan")),
                                       ("K", float("inf")), ("K", float("-inf"))])
def test_any_span_length_keeps_what_is_not_finite_to_the_rows_that_attend_it(which, bad, span, form):
    """A K or V row that is not finite reaches the rows that attend it and no others, as in the row-stationary
    form.  (An infinite key leaves those rows finite whose score it sends to -inf.)"""
    Hq, Hkv, L, D, S, k, q0 = 8, 2, 6000, 128, 77, 8, 2000
    Q, K, V = make(801, Hq, Hkv, L, D, torch.bfloat16, Lq=L - q0, scale=1.0 if form == "joint" else 0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0, want_scores=True)
    assert takes_matrix_cores(Q, K, S, k, q0)
    t = S * span + 30
    (K if which == "K" else V)[0, t, 5] = bad
    if form == "joint":
        O, R = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0)[0], row_form(Q, K, V, idx, None, S, q0)[0]
    else:
        O = B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, q_pos0=q0)
        R = row_form(Q, K, V, idx, sc, S, q0)
    torch.cuda.synchronize()
    finite = torch.isfinite(O.float()).all(dim=2)
    assert torch.equal(finite, torch.isfinite(R.float()).all(dim=2))
    pos = q0 + torch.arange(L - q0, device=DEV)
    attends = (idx == t // S).any(dim=2) | ((pos // S == t // S) & (pos >= t))[None, :]
    attends[Hq // Hkv:] = False
    if which == "V" or math.isnan(bad):
        assert torch.equal(~finite, attends)
    else:
        assert not bool((~finite & ~attends).any())


@pytest.mark.parametrize("form,dtype,Hq,Hkv,S,A,k,nb", [
    ("joint", torch.bfloat16, 32, 4, 512, 512, 16, 2),    # 128-token chunks: one batch of rows, kept in registers
    ("gated", torch.float32, 16, 2, 512, 512, 16, 2),     # the same in fp32: 64-token chunks
    ("anchor", torch.bfloat16, 32, 4, 1, 1, 8, 2),        # and where spans cover parts of a chunk
    ("joint", torch.bfloat16, 16, 2, 1024, 1024, 16, 8),  # 512-token chunks: read again
    ("joint", torch.bfloat16, 24, 8, 512, 256, 16, 8),    # overlapping spans: every entry its own range
    ("gated", torch.float32, 16, 2, 600, 600, 16, 8),     # a second, shorter chunk
])
def test_decode_entries_sharing_chunks_go_in_pairs(form, dtype, Hq, Hkv, S, A, k, nb):
    """Steps of 224 MB and more of routed rows pair the entries that share a chunk: a batch of the same
    sequence (256 MB and more) against the single step (157 MB at most: every entry by itself).  Heads list the
    same spans, partly the same, an odd number of them, and empty slots.  Chunks may be cut differently: fp32
    sums in another order (1e-5 of outputs below 5), then one rounding to the output's type."""
    D, G = 128, Hq // Hkv
    routed = Hq * k * (1201 if form == "anchor" else S) * 2 * D * (2 if dtype == torch.bfloat16 else 4)
    assert routed <= 160 << 20 and nb * routed >= 256 << 20
    rng = np.random.default_rng(S + k)
    L = 40000 if form == "anchor" else max(S * 22, 9000) + 37
    Q, K, V = make(900 + S, Hq, Hkv, L, D, dtype, Lq=1, scale=0.5)
    if form == "anchor":
        from tests.test_parity_gpu import clustered_anchors
        idx = clustered_anchors(rng, L - 1, 1088, 2, Hkv, G, k)
    else:
        c = (L - 1) // A
        idx = np.full((Hq, 1, k), -1, np.int32)
        for h in range(Hq):
            common = np.random.default_rng(h // G).choice(c, size=k, replace=False)
            own = rng.choice(c, size=k, replace=False)
            pick = common if h % G in (0, 2, 3) else np.unique(np.concatenate([common[:k // 2], own]))[:k] if h % 2 else own
            pick = np.sort(pick)[: k - (h % 3)]
            idx[h, 0, :len(pick)] = pick
    sc = rng.standard_normal((Hq, 1, k)).astype(np.float32)
    idx_t, sc_t = torch.from_numpy(idx).to(DEV), torch.from_numpy(sc).to(DEV)
    stride = 0 if A == S else A
    batch = B.DecodeBatch([Q] * nb, [Q] * nb, [K] * nb, [V] * nb, None, S, k, want_scores=True, span_stride=stride)
    batch.idx.copy_(idx_t.expand(nb, -1, -1, -1))
    batch.scores.copy_(sc_t.expand(nb, -1, -1, -1))
    if form == "anchor":
        one = B.sl_anchor_attention_decode(Q, K, V, idx_t, sc_t, 1088, 4, 2)
        many = B.sl_anchor_attention_decode_batched(batch, 1088, 4, 2)
    elif form == "gated":
        one = B.sl_span_attention_combined_decode(Q, K, V, idx_t, sc_t, S, span_stride=stride)
        many = B.sl_span_attention_combined_decode_batched(batch)
    else:
        one, lse = B.sl_span_attention_decode(Q, K, V, idx_t, S, span_stride=stride)
        many, lses = B.sl_span_attention_decode_batched(batch)
        torch.cuda.synchronize()
        assert float((lses - lse).abs().max()) <= 1e-5
    torch.cuda.synchronize()
    step = 2 ** -7 if dtype == torch.bfloat16 else 0.0
    diff = (many.float() - one.float()[None]).abs() - step * one.float().abs()[None]
    assert float(diff.max()) <= 1e-5


@pytest.mark.parametrize("Hq,Hkv,D,L,k,w,root,Lq,q0", [
    (8, 1, 128, 700, 2, 0, 2, None, 0),          # rows with no candidate, with one, with a batch and a remainder
    (12, 1, 64, 3001, 4, 24, 2, 1501, 1500),     # more than 8 heads a group, D = 64, odd row count
    (4, 4, 128, 40000, 8, 255, 2, 9, 39991),     # one head a group, many batches, lists of 8
    (6, 2, 128, 9000, 3, 8, 3, 1030, 7970),      # cubes; rows past one chunk of the block order
    (8, 2, 128, 20, 2, 1088, 2, None, 0),        # no row has a candidate
    # the same where the rows have candidates enough for the matrix cores
    (8, 1, 128, 8500, 2, 0, 2, None, 0),
    (8, 2, 128, 2603, 2, 0, 2, None, 0),         # every count from 0 to 50, pairs of rows on both sides of a batch's end
    (8, 2, 128, 14001, 4, 0, 2, None, 0),
    (12, 1, 64, 30001, 4, 24, 2, 1501, 28500),
    (4, 4, 128, 40000, 3, 255, 2, 9, 39991),
    (6, 1, 128, 600000, 3, 8, 3, 17001, 582999),
])
def test_anchor_search_on_the_matrix_cores(Hq, Hkv, D, L, k, w, root, Lq, q0):
    """Batches of 16 candidates, pairs of rows and the lists' merge against fp64 scores: the selection by the
    tie margin of the search tests, the scores to 1e-4 (fp32 sums of up to 128 exact products below 10)."""
    from tests.test_parity_gpu import check_anchor_row
    Q, K, _ = make(1000 + L, Hq, Hkv, L, D, torch.bfloat16, Lq=Lq, scale=0.5)
    an, sc = B.sl_anchor_search_prefill(Q, K, k, w, q_pos0=q0, want_scores=True, search_root=root)
    torch.cuda.synchronize()
    Qn, Kn, an, sc = f64(Q), f64(K), an.cpu().numpy(), sc.cpu().numpy()
    G, n = Hq // Hkv, Q.shape[1]
    for h in range(Hq):
        for r in sorted({0, 1, 2, 3, n // 2, n - 2, n - 1, *range(0, n, 97)}):
            if not 0 <= r < n:
                continue
            cand = orc.anchor_candidates(q0 + r, w, root)
            s = np.array([float(Qn[h, r] @ Kn[h // G, t]) for _, t in cand])
            order = sorted(np.lexsort((np.arange(len(s)), -s))[:k].tolist())
            want = [cand[j][1] for j in order] + [-1] * (k - len(order))
            check_anchor_row(an[h, r].tolist(), want, cand, s, k, (h, r))
            of = {t: x for (_, t), x in zip(cand, s)}
            for t, x in zip(an[h, r], sc[h, r]):
                assert (t < 0 and x == -np.inf) or abs(x - of[t]) <= 1e-4


def test_anchor_search_ties_go_to_the_nearer_anchor():
    """Every key one of three rows: nearly all candidates tie, across the four lanes of a column."""
    L, k, w = 30000, 4, 24
    Q, K, _ = make(1101, 8, 1, L, 128, torch.bfloat16, Lq=3)
    base = K[0, :3].clone()
    K[0] = base[torch.arange(L, device=DEV) % 3]
    an, sc = B.sl_anchor_search_prefill(Q, K, k, w, q_pos0=L - 3, want_scores=True)
    torch.cuda.synchronize()
    an = an.cpu().numpy()
    for r in range(3):
        i = L - 3 + r
        toks = np.array([t for _, t in orc.anchor_candidates(i, w, 2)])
        s3 = f64(Q[:, r]) @ f64(base).T
        for h in range(8):
            s = s3[h][toks % 3]
            pick = np.sort(np.lexsort((np.arange(len(s)), -s))[:k])
            assert an[h, r].tolist() == toks[pick].tolist()


@pytest.mark.parametrize("kind", ["random", "cancelling", "near-equal", "zero", "infinite", "nan", "huge"])
@pytest.mark.parametrize("Hq,Hkv,D,k", [(8, 1, 128, 2), (6, 2, 128, 4), (12, 1, 64, 3), (8, 2, 128, 6)])
def test_anchor_search_selects_as_the_decode_search_does(Hq, Hkv, D, k, kind):
    """Whatever the scores: the selection and the returned scores of every row are the decode search's to the
    bit, and do not depend on how a prompt is cut.  Cancelling: two large channels of opposite sign, so that the
    order of the additions decides between scores.  Near-equal: three keys, each varying in one small element.  Zero: queries and stretches of keys that are all zero.  Infinite, nan: keys that are not
    finite among finite ones, one and many.  Huge: scores around 1e38, where no number may take the place of their low bits."""
    L, q0, w = 27000, 25000, 24
    Q, K, _ = make(1300 + D + k, Hq, Hkv, L, D, torch.bfloat16, Lq=L - q0, scale=0.3)
    if kind == "cancelling":
        Q[..., 3], Q[..., D - 20] = 61.0, -61.0
        K[..., 3] = K[..., D - 20] = (40 + 20 * torch.rand(K.shape[:2], device=DEV)).to(torch.bfloat16)
    elif kind == "near-equal":
        K.copy_(K[:, :3].clone()[:, torch.arange(L, device=DEV) % 3])
        K[..., 5] = (2.0 ** -13 * torch.randn(K.shape[:2], device=DEV)).to(torch.bfloat16)
    elif kind == "zero":
        Q[:, 1::3] = 0
        K[:, 5000:12000] = 0
    elif kind == "huge":
        Q.mul_(3e18)
        K.mul_(3e18)
    elif kind == "infinite":
        K[0, 12000, 7], K[0, 11000, 7] = float("inf"), float("-inf")
    elif kind == "nan":
        K[0, 12000, 7] = float("nan")
        K[Hkv - 1, 14000:20000:3, D - 1] = float("nan")
    an, sc = B.sl_anchor_search_prefill(Q, K, k, w, q_pos0=q0, want_scores=True)
    only = B.sl_anchor_search_prefill(Q, K, k, w, q_pos0=q0)
    parts = [B.sl_anchor_search_prefill(Q[:, a:b], K[:, :q0 + b], k, w, q_pos0=q0 + a, want_scores=True)
             for a, b in ((0, 1), (1, 500), (500, 1277), (1277, L - q0))]
    torch.cuda.synchronize()
    assert torch.equal(an, only)
    assert torch.equal(an, torch.cat([p[0] for p in parts], dim=1))
    assert torch.equal(sc.view(torch.int32), torch.cat([p[1] for p in parts], dim=1).view(torch.int32))
    for r in sorted({0, L - q0 - 1, L - q0 - 2, *range(1, L - q0, 41)}):
        da, ds = B.sl_anchor_search_decode(Q[:, r:r + 1], K[:, :q0 + r + 1], k, w, want_scores=True)
        torch.cuda.synchronize()
        assert torch.equal(da[:, 0], an[:, r]), r
        assert torch.equal(ds[:, 0].view(torch.int32), sc[:, r].view(torch.int32)), r


@pytest.mark.parametrize("k,scores", [(1, False), (4, True), (5, False), (8, True), (9, False)])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 97])
def test_prefill_search_stages_and_list_lengths(n, k, scores):
    """Candidate counts around the 32-key stages for every list length's instantiation, keys packed and read
    from the cache, against the oracle."""
    from tests.test_parity_gpu import check_idx
    S = 4
    L = S * n + 2
    Q, K, _ = make(1200 + n, 4, 2, L, 128, torch.bfloat16)
    Ks = B.sl_span_keys(K, S)
    r = B.sl_span_search_prefill(Q, K, Ks, S, k, want_scores=scores)
    idx = r[0] if scores else r
    again = B.sl_span_search_prefill(Q, K, None, S, k)
    torch.cuda.synchronize()
    assert torch.equal(idx, again)
    rows = [(h, r) for h in range(4) for r in sorted({0, S - 1, S, L // 2, L - 2, L - 1, *range(0, L, 13)}) if r < L]
    check_idx(idx, Q, Ks, S, k, 0, rows)
    if scores:
        q, kn, sc, ix = f64(Q), f64(Ks), r[1].cpu().numpy(), idx.cpu().numpy()
        for h, row in rows:
            for j, x in zip(ix[h, row], sc[h, row]):
                assert (j < 0 and x == -np.inf) or abs(x - q[h, row] @ kn[h // 2, j]) <= 1e-3


@pytest.mark.parametrize("n,k", [(31, 5), (32, 8), (33, 1), (64, 16), (257, 8), (500, 4), (1025, 4), (2050, 4),
                                 (4096, 8), (4097, 8), (300, 32)])
@pytest.mark.parametrize("kind", ["levels", "pairs", "equal", "zeros", "negative", "masked", "infinite", "nan"])
def test_prefill_search_scores_that_agree_in_their_leading_bits(n, k, kind):
    """Scores that differ only in the bits whose place the span's number takes, in twos and in longer runs around the
    k-th; all alike; nothing but zeros around the k-th, a few scores above them; keys masked with -inf in one channel; out of
    range.  Whole numbers below 2^24: products and sums are exact, the oracle decides, to the index.  What is not
    finite has no oracle: the form that returns scores carries none of the numbers."""
    S, Lq, Hq, Hkv, D = 2, 200, 4, 2, 128
    L = S * n + S - 1
    Lq = min(Lq, L)
    g = torch.Generator().manual_seed(n * 100 + k)
    K = torch.zeros((Hkv, L, D))
    Q = torch.zeros((Hq, Lq, D))
    Q[:, :, 0], Q[:, :, 1] = 4096.0, 1.0
    Q[:, :, 2] = torch.randint(-2, 3, (Hq, Lq), generator=g).float()
    j = torch.randperm(n, generator=g).float()
    if kind == "levels":        # a few leading parts, all of them with many different low parts
        K[:, 1::2, 0], K[:, 1::2, 1] = (j % 7) + 64, torch.floor(j / 7) % 100
        K[:, 1::2, 2] = (j % 3) - 1
    elif kind == "pairs":       # every leading part twice, the low part decides (or nothing does)
        lead = torch.floor(j / 2)
        K[:, 1::2, 0], K[:, 1::2, 3] = lead % 128 + 1, torch.floor(lead / 128)
        Q[:, :, 3] = 128 * 4096.0
        K[:, 1::2, 1] = torch.where(lead % 3 == 0, torch.zeros(n), j % 2)
    elif kind == "equal":
        K[:, 1::2, 1] = 3.0
        Q[:, :, 2] = 0.0
    elif kind == "zeros":
        K[:, 1::2, 1] = torch.where(j < 3, j + 1, torch.where(j % 4 == 0, -1.0 - j % 7, torch.zeros(n)))
        Q[:, :, 2] = 0.0
    elif kind in ("negative", "masked"):
        K[:, 1::2, 0], K[:, 1::2, 1] = -((j % 5) + 64), torch.floor(j / 5) % 100
        if kind == "masked":
            Q[:, :, 4] = 1.0
            K[:, 1::2, 4] = torch.where(j % 3 == 0, torch.full((n,), float("-inf")), torch.zeros(n))
    else:
        K[:, 1::2, 0] = torch.randn((Hkv, n), generator=g)
        K[:, 1::2, 1] = torch.randn((Hkv, n), generator=g)
        some = torch.rand((Hkv, n), generator=g) < 0.1
        if kind == "infinite":
            K[:, 1::2, 0] = torch.where(some, torch.sign(K[:, 1::2, 0]) * 3e38, K[:, 1::2, 0])
        else:
            K[:, 1::2, 5] = torch.where(some, torch.full((Hkv, n), float("nan")), torch.zeros(Hkv, n))
    Q, K = Q.to(torch.bfloat16).to(DEV), K.to(torch.bfloat16).to(DEV)
    q0 = L - Lq
    idx = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0)
    two, _ = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0, want_scores=True)
    torch.cuda.synchronize()
    if kind != "nan":
        assert torch.equal(idx, two)
    if kind in ("infinite", "nan"):
        ok = ((idx >= -1) & (idx < n)).all()
        assert bool(ok)
        return
    Qn, Kn, got = f64(Q), f64(B.sl_span_keys(K, S)), idx.cpu().numpy()
    for h in range(Hq):
        for r in sorted({0, 1, Lq // 2, Lq - 2, Lq - 1, *range(0, Lq, 17)}):
            s = orc.search_scores_row(Qn[h, r], Kn[h // 2], (q0 + r) // S)
            if np.isfinite(s).sum() < min(k, len(s)):
                continue    # a masked span is chosen for want of others: equal to the form that returns scores, above
            want = orc.select_topk(s, k)
            assert got[h, r].tolist() == want + [-1] * (k - len(want)), (h, r)


@pytest.mark.parametrize("n", [7, 300, 900])     # one launch, one launch of several loads, two launches
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_decode_search_writes_every_slot_where_scores_are_minus_infinity(n, dtype):
    """Fewer finite scores than slots: the candidates with one are selected, the other slots say that they are empty,
    whatever the output held; single and batched, grid and anchors."""
    S, k, Hq, Hkv, D = 3, 10, 4, 2, 128
    L = S * n + 2
    Q, K, V = make(3450 + n, Hq, Hkv, L, D, dtype, Lq=1)
    Q[..., 3] = 1.0
    left = sorted({0, n // 2, n - 1})
    K[:, :, 3] = float("-inf")
    for j in left:
        K[:, S * (j + 1) - 1, 3] = 0.0
    p = B.make_params(Q, K, S, k, L - 1)
    ws, stream = B.Workspace(), torch.cuda.current_stream().cuda_stream
    wptr, wbytes = ws.get(B.workspace_bytes(p, B.OP_SEARCH_DECODE))
    idx = torch.full((Hq, 1, k), 5, dtype=torch.int32, device=DEV)
    sc = torch.full((Hq, 1, k), 5.0, device=DEV)
    assert B.load().sl_span_search_decode(ctypes.byref(p), Q.data_ptr(), K.data_ptr(), None, idx.data_ptr(), sc.data_ptr(),
                                          wptr, wbytes, stream) == B.SL_OK
    bt = B.DecodeBatch([Q, Q], [Q, Q], [K, K], [V, V], None, S, k, want_scores=True)
    bt.idx.fill_(5), bt.scores.fill_(5.0)
    B.sl_span_search_decode_batched(bt)
    anchors = torch.full((Hq, 1, k), 5, dtype=torch.int32, device=DEV)
    pa, g = B.make_params(Q, K, 1, k, L - 1), B.SlAnchorGeometry(0, 0, 0, 2, 0)
    assert B.load().sl_anchor_search_decode(ctypes.byref(pa), ctypes.byref(g), Q.data_ptr(), K.data_ptr(), anchors.data_ptr(),
                                            None, stream) == B.SL_OK
    torch.cuda.synchronize()
    for i, s in ((idx, sc), (bt.idx[0], bt.scores[0]), (bt.idx[1], bt.scores[1])):
        assert i[:, 0].tolist() == [left + [-1] * (k - len(left))] * Hq
        assert bool(torch.isfinite(s[:, 0, :len(left)]).all()) and bool((s[:, 0, len(left):] == float("-inf")).all())
    # anchors i - (s + 1)^2 + 1 whose keys are not masked, the nearest first
    near = [t for t in (L - (x + 1) ** 2 for x in range(L)) if t >= 0 and bool(torch.isfinite(K[0, t, 3]))]
    assert anchors[:, 0].tolist() == [near[:k] + [-1] * (k - len(near))] * Hq


def test_prefill_search_of_equal_scores_takes_two_walks():
    """Two walks over the candidates, not three: 1.85 times the time of scores that differ (three: 2.5)."""
    L, S, k = 20000, 128, 8
    Q, K, _ = make(3400, 32, 4, L, 128, torch.bfloat16)
    flat = K[:, :1].expand(-1, L, -1).contiguous()
    took = []
    for keys in (K, flat):
        Ks = B.sl_span_keys(keys, S)
        for _ in range(3):
            idx = B.sl_span_search_prefill(Q, keys, Ks, S, k)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times = []
        for _ in range(7):
            ev[0].record()
            for _ in range(20):
                B.sl_span_search_prefill(Q, keys, Ks, S, k)
            ev[1].record()
            torch.cuda.synchronize()
            times.append(ev[0].elapsed_time(ev[1]))
        took.append(sorted(times)[3])
    assert idx[0, L - 1].tolist() == list(range(k))
    assert took[1] <= 2.15 * took[0], took


F32 = [
    # Hq Hkv L   D    S    A    k  form     q_pos0 Lq
    (4, 4, 2500, 64, 64, 64, 4, "joint", 0, 2500),
    (4, 1, 3000, 64, 55, 55, 4, "gated", 0, 3000),         # windows that start inside a tile of 16 rows
    (8, 2, 2600, 128, 39, 39, 9, "joint", 600, 1999),      # a list that is no whole number of slots at a time
    (4, 2, 5000, 64, 81, 81, 8, "joint", 0, 5000),         # a row more than is staged at a time
    (4, 4, 4000, 128, 65, 65, 3, "gated", 1001, 2999),
    (8, 8, 3001, 64, 142, 142, 5, "joint", 0, 3001),
    (8, 1, 4000, 64, 128, 64, 8, "gated", 0, 4000),        # overlapping spans, each its own softmax
    (16, 1, 2500, 64, 80, 80, 17, "joint", 0, 2500),
]


def span_rows(Q, K, V, idx, sc, S, q0, stride):
    """(this form, the row-stationary form) of a call, O first."""
    if sc is None:
        return (B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0, span_stride=stride),
                row_form(Q, K, V, idx, None, S, q0, stride))
    return ((B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, q_pos0=q0, span_stride=stride),),
            (row_form(Q, K, V, idx, sc, S, q0, stride),))


@pytest.mark.parametrize("Hq,Hkv,L,D,S,A,k,form,q_pos0,Lq", F32)
def test_fp32_spans_on_the_matrix_cores(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq):
    """fp32 tiles against the row-stationary kernels, packed and strided.  Both round some hundred sums of fp32 products
    (2^-24 each, of terms below 5): outputs below 5 agree to 2^-24 * 5 * sqrt(700) * 2 = 1.6e-5, and are not all equal,
    which they would be if the same kernels had run twice."""
    stride = 0 if A == S else A
    Q, K, V = make(2000 + L + S, Hq, Hkv, L, D, torch.float32, Lq=Lq, scale=1.0 if form == "joint" else 0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, A, k, q_pos0=q_pos0, want_scores=True)
    sc = None if form == "joint" else torch.where(torch.isfinite(sc), sc, 0.0)
    assert takes_matrix_cores(Q, K, S, k, q_pos0, stride)
    got, want = span_rows(Q, K, V, idx, sc, S, q_pos0, stride)
    strided, _ = span_rows(token_major(Q), token_major(K), token_major(V), idx, sc, S, q_pos0, stride)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(got, strided))
    assert float((got[0] - want[0]).abs().max()) <= 1.6e-5
    assert not torch.equal(got[0], want[0])
    if form == "joint":
        assert float((got[1] - want[1]).abs().max()) <= 1e-5
        check_attention(*got, Q, K, V, idx, S, q_pos0, 0.0, [(h, r) for h in range(Hq) for r in range(0, Lq, 397)], stride=stride or None)


@pytest.mark.parametrize("form", ["joint", "gated"])
def test_fp32_spans_in_several_passes_over_the_kv_heads(form):
    """More partials than 4 GiB of scratch hold: three kv heads, then the fourth, in the same workspace; packed and strided.
    The sums' bound is that of test_fp32_spans_on_the_matrix_cores."""
    Hq, Hkv, L, D, S, k = 32, 4, 19411, 128, 64, 16
    Q, K, V = make(2060, Hq, Hkv, L, D, torch.float32, scale=1.0 if form == "joint" else 0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, want_scores=True)
    sc = None if form == "joint" else torch.where(torch.isfinite(sc), sc, 0.0)
    need = B.workspace_bytes(B.make_params(Q, K, S, k), B.OP_ATTENTION_PREFILL)
    assert 3 * Hq // Hkv * L * k * D * 4 < need < Hq * L * k * D * 4
    got, want = span_rows(Q, K, V, idx, sc, S, 0, 0)
    torch.cuda.synchronize()
    for x, y in zip(got, want):
        assert float((x - y).abs().max()) <= 1.6e-5
    for kv in range(Hkv):       # all of them by this form
        heads = slice(kv * Hq // Hkv, (kv + 1) * Hq // Hkv)
        assert not torch.equal(got[0][heads], want[0][heads]), kv
    del want
    strided = B.sl_span_attention_prefill(token_major(Q), token_major(K), token_major(V), idx, S)[0] if sc is None else \
        B.sl_span_attention_combined_prefill(token_major(Q), token_major(K), token_major(V), idx, sc, S)
    torch.cuda.synchronize()
    assert torch.equal(got[0], strided)


@pytest.mark.parametrize("form", ["joint", "gated"])
@pytest.mark.parametrize("span", [12, 50])     # a span that lies in no row's window; one that does
@pytest.mark.parametrize("which,bad", [("V", float("nan")), ("V", float("inf")), ("K", float("nan")), ("K", float("inf"))])
def test_fp32_spans_keep_what_is_not_finite_to_the_rows_that_attend_it(which, bad, span, form):
    Hq, Hkv, L, D, S, k, q0 = 8, 2, 4200, 64, 61, 8, 1500
    Q, K, V = make(2100, Hq, Hkv, L, D, torch.float32, Lq=L - q0, scale=1.0 if form == "joint" else 0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0, want_scores=True)
    assert takes_matrix_cores(Q, K, S, k, q0)
    t = S * span + 30
    (K if which == "K" else V)[0, t, 5] = bad
    got, want = span_rows(Q, K, V, idx, None if form == "joint" else sc, S, q0, 0)
    torch.cuda.synchronize()
    finite = torch.isfinite(got[0]).all(dim=2)
    assert torch.equal(finite, torch.isfinite(want[0]).all(dim=2))
    pos = q0 + torch.arange(L - q0, device=DEV)
    attends = (idx == t // S).any(dim=2) | ((pos // S == t // S) & (pos >= t))[None, :]
    attends[Hq // Hkv:] = False
    assert not bool((~finite & ~attends).any())
    assert bool((~finite).any())


MASKED = [
    # D  S    first and last masked key of the span
    (64, 64, 0, 64),        # a whole span of one stage
    (64, 142, 0, 80),       # the first of two stages (80 rows at D = 64), exactly
    (64, 142, 0, 79), (64, 142, 0, 142), (64, 142, 80, 142),
    (128, 65, 0, 64),       # ... (64 at D = 128): one key is left
    (128, 65, 0, 65),
]


@pytest.mark.parametrize("D,S,lo,hi,form,how", [(*m, f, how) for m in MASKED for f in ("joint", "gated") for how in ("masked", "overflow")]
                         + [(*m, "gated", "values") for m in MASKED if m[2:] == (0, m[1])])
def test_fp32_spans_whose_scores_are_all_minus_infinity(D, S, lo, hi, form, how):
    """Keys masked with -inf in one channel, or finite ones whose products overflow to it, or masked ones beside values
    that are infinite (in the gated form, where the row form too meets a span's values by themselves): what is left of the
    span counts, a span of which nothing is left has no weight, and no row becomes NaN by it; in slots and in windows;
    against the row-stationary kernels.  The sums' bound is that of test_fp32_spans_on_the_matrix_cores."""
    Hq, Hkv, L, k, span = 8, 2, 4200, 4, 7
    q0 = span * S + S // 2      # the first rows' window is the span's, and in the middle of it
    Q, K, V = make(2150 + S, Hq, Hkv, L, D, torch.float32, Lq=L - q0, scale=1.0 if form == "joint" else 0.35)
    Q[:, :, 5] = Q[:, :, 5].abs() + 0.1
    K[:, :, 5] = 0
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0, want_scores=True)
    lists = (idx == span).any(dim=2)
    takes = ~lists & ((q0 + torch.arange(L - q0, device=DEV)) // S > span)[None, :]
    takes[:, 1::2] = False
    takes[0] = False
    for h in range(Hq):         # in every slot, the first and the last among them
        idx[h, :, h % k] = torch.where(takes[h], span, idx[h, :, h % k])
    assert takes_matrix_cores(Q, K, S, k, q0)
    at = slice(S * span + lo, S * span + hi)
    if how == "overflow":
        Q[:, :, 5] *= 1e20
        K[:, at, 5] = -1e22
    else:
        K[:, at, 5] = float("-inf")
    if how == "values":
        V[:, at, 3] = float("inf")
    got, want = span_rows(Q, K, V, idx, None if form == "joint" else sc, S, q0, 0)
    torch.cuda.synchronize()
    for x, y in zip(got, want):
        ok = torch.isfinite(y)
        assert torch.equal(torch.isfinite(x), ok)
        assert float(torch.where(ok, x - y, 0.0).abs().max()) <= 1.6e-5
    later = slice(S, None)      # rows whose window holds none of the masked keys
    assert bool(torch.isfinite(got[0][:, later]).all())
    assert bool(takes[:, later].any()) and bool((idx[:, later] == span).any())


@pytest.mark.parametrize("form", ["joint", "gated"])
@pytest.mark.parametrize("repeats", [0, 1, 4])
def test_fp32_rows_that_list_a_span_twice_cost_no_other_row_its_span(repeats, form):
    """Chunks whose every row lists one span fill its list of rows to the last place; some rows that list it in several
    slots (their own result is unspecified) leave the others as they are, in a workspace that holds NaN."""
    Hq, Hkv, L, D, S, k, Lq = 8, 1, 64 * 264, 64, 64, 4, 512     # two chunks of 256 rows x 8 heads
    q0 = L - Lq
    Q, K, V = make(2170, Hq, Hkv, L, D, torch.float32, Lq=Lq, scale=1.0 if form == "joint" else 0.35)
    g = torch.Generator().manual_seed(repeats)
    idx = torch.stack([torch.randperm(250, generator=g)[:k] for _ in range(Hq * Lq)]).to(torch.int32).reshape(Hq, Lq, k)
    idx = torch.where(idx == 77, 251, idx)
    idx[:, :, 2] = 77
    bad = torch.zeros((Hq, Lq), dtype=torch.bool)
    if repeats:
        bad[:, 100::200] = True
        idx[:, 100::200, :repeats] = 77
    idx, bad = idx.to(DEV), bad.to(DEV)
    sc = None if form == "joint" else torch.randn((Hq, Lq, k), generator=g).to(DEV)
    assert takes_matrix_cores(Q, K, S, k, q0)
    ws = B.Workspace()
    ws.get(B.workspace_bytes(B.make_params(Q, K, S, k, q0), B.OP_ATTENTION_PREFILL))
    ws.buf.fill_(255)
    if form == "joint":
        got, want = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0, ws=ws)[0], row_form(Q, K, V, idx, None, S, q0)[0]
    else:
        got, want = B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, q_pos0=q0, ws=ws), row_form(Q, K, V, idx, sc, S, q0)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(got).all())
    assert float((got - want)[~bad].abs().max()) <= 1.6e-5     # the bound of test_fp32_spans_on_the_matrix_cores


def test_fp32_overlapping_spans_in_one_softmax_take_no_scratch():
    """They go through the row-stationary kernels whatever scratch there is, so the call allocates its outputs only; the
    gated form of the same shape, which does not, allocates partials."""
    Hq, Hkv, L, D, S, A, k = 8, 1, 4000, 64, 128, 64, 8
    Q, K, V = make(2180, Hq, Hkv, L, D, torch.float32, scale=0.35)
    idx, sc = B.sl_span_search_prefill(Q, K, None, A, k, want_scores=True)
    sc = torch.where(torch.isfinite(sc), sc, 0.0)
    assert takes_matrix_cores(Q, K, S, k, 0, A)
    partials = Hq * L * k * D * 4
    grown = []
    for call in (lambda: B.sl_span_attention_prefill(Q, K, V, idx, S, span_stride=A),
                 lambda: B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, span_stride=A)):
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        out = call()
        torch.cuda.synchronize()
        grown.append(torch.cuda.max_memory_allocated() - before)
        del out
    assert grown[0] < 2 * Hq * L * (D + 1) * 4 < partials < grown[1]


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (3, 1), (6, 1), (12, 2), (8, 1), (16, 1)])
@pytest.mark.parametrize("Lq,S", [(1, 64), (15, 64), (17, 192), (129, 128), (200, 77)])
def test_window_tiles_of_several_heads(Hq, Hkv, Lq, S):
    """Groups of 1, 3, 6, 8 and 16 heads: 1, 2 and 8 heads of a window tile, row counts around a tile's 128, 64 and 16
    rows, with the merge in the window kernel and behind it, spans of any length, and the sliding window; against the
    oracle and the row-stationary form."""
    from tests.test_parity_gpu import check_combined
    L, k = 64 * 30 + 11, 3
    q0 = L - Lq
    Q, K, V = make(2200 + Hq + Lq, Hq, Hkv, L, 128, torch.bfloat16, Lq=Lq, scale=0.5)
    idx, sc = B.sl_span_search_prefill(Q, K, None, S, k, q_pos0=q0, want_scores=True)
    O, LSE = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0)
    C = B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, q_pos0=q0)
    an, asc = B.sl_anchor_search_prefill(Q, K, 2, 120, q_pos0=q0, want_scores=True)
    A = B.sl_anchor_attention_prefill(Q, K, V, an, asc, 120, 2, 1, q_pos0=q0)
    R = B.sl_anchor_attention_prefill(Q, K, V, an, asc, 120, 2, 1, q_pos0=q0, row_stationary=True)
    torch.cuda.synchronize()
    rows = [(h, r) for h in range(Hq) for r in sorted({0, 1, Lq // 2, Lq - 1, *range(0, Lq, 37)}) if r < Lq]
    check_attention(O, LSE, Q, K, V, idx, S, q0, 0.0, rows)
    check_combined(C, Q, K, V, idx, sc, S, q0, 0.0, rows)
    assert float((A.float() - R.float()).abs().max()) <= 3e-2    # the bound of the masked kv tiles' test


@pytest.mark.parametrize("form", ["joint", "gated"])
@pytest.mark.parametrize("D,S", [(128, 65), (128, 128), (128, 200), (128, 320), (64, 137), (64, 300)])
def test_decode_batches_of_many_short_spans(D, S, form):
    """Items enough for every chunk length (8 x 32 x 17): chunks of 128 and 256 tokens that spans fill badly, exactly and
    with a remainder, against the single-sequence entry points.  Other chunks add in another order: outputs differ by a
    rounding to bf16, 2^-7 of them, and what fp32 sums of some thousand terms differ by."""
    gated = form == "gated"
    seqs = [make(2300 + S + b, 32, 4, S * 18 + 700 - 83 * b, D, torch.bfloat16, Lq=1, scale=0.5) for b in range(8)]
    Q, K, V = ([s[x] for s in seqs] for x in range(3))
    bt = B.DecodeBatch(Q, Q, K, V, [B.sl_span_keys(k, S) for k in K], S, 16, want_scores=gated)
    if gated:
        idx, sc = B.sl_span_search_decode_batched(bt)
        O = B.sl_span_attention_combined_decode_batched(bt)
    else:
        idx = B.sl_span_search_decode_batched(bt)
        O, LSE = B.sl_span_attention_decode_batched(bt)
    for b in range(8):
        if gated:
            i1, s1 = B.sl_span_search_decode(Q[b], K[b], None, S, 16, want_scores=True)
            o1 = B.sl_span_attention_combined_decode(Q[b], K[b], V[b], i1, s1, S)
        else:
            i1 = B.sl_span_search_decode(Q[b], K[b], None, S, 16)
            o1, l1 = B.sl_span_attention_decode(Q[b], K[b], V[b], i1, S)
        torch.cuda.synchronize()
        assert torch.equal(idx[b], i1)
        assert float(((O[b].float() - o1.float()).abs() - 2 ** -7 * o1.float().abs()).max()) <= 1e-5
        if not gated:
            assert float((LSE[b] - l1).abs().max()) <= 1e-5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [0, 1])
def test_decode_steps_on_both_sides_of_one_launch(D, rows):
    """160 KB of K a head (and a row more) in slots of several sizes and forms: spans of a wavefront's load and less, more
    and with a remainder, spans that overlap, empty and foreign slots, no slot at all."""
    limit = 80 * 1024 // D
    for S, A, k in ((limit // 5 + rows, limit // 5 + rows, 4), (limit // 33 + rows, limit // 33 + rows, 32),
                    (limit + rows, limit + rows, 0), (limit // 2 + rows, (limit // 2 + rows) // 3, 1),
                    (limit // 10 + rows, (limit // 10 + rows + 1) // 2, 9), (7, 7, 5), (1, 1, 2)):
        L = A * (k + 9) + S + 1
        Q, K, V = make(3100 + S + k, 8, 2, L, D, torch.bfloat16, Lq=1)
        c = (L - 1) // A
        g = torch.Generator().manual_seed(S)
        idx = torch.stack([torch.randperm(c, generator=g)[:k] for _ in range(8)]).to(torch.int32).reshape(8, 1, k)
        if k > 1:
            idx[1, 0, 0], idx[2, 0, k - 1], idx[3, 0, 1], idx[4] = -1, c, 10 ** 6, -1
        idx = idx.to(DEV)
        O, LSE = B.sl_span_attention_decode(Q, K, V, idx, S, span_stride=A)
        torch.cuda.synchronize()
        check_attention(O, LSE, Q, K, V, idx, S, L - 1, 0.0, stride=A)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L,S,k", [(3000, 33, 32), (16411, 128, 8), (20000, 100, 8), (100000, 320, 16)])
def test_fp32_decode_steps_against_64_bits(D, L, S, k):
    """Chunks of 64 and 128 tokens: products and sums in fp32 throughout.  A weighted mean of some hundred to some thousand
    terms, added up in parts of at most 32, has a relative error of a few times 2^-24 over all outputs (measured 1.6e-7 to
    2.0e-7); 2^-22 is where a sum has gone through one part too long."""
    Hq, Hkv = 32, 4
    Q, K, V = make(3240 + S, Hq, Hkv, L, D, torch.float32, Lq=1)
    idx = B.sl_span_search_decode(Q, K, None, S, k)
    O, LSE = B.sl_span_attention_decode(Q, K, V, idx, S)
    c = (L - 1) // S
    exact, lse = torch.empty((Hq, D), dtype=torch.float64), torch.empty(Hq, dtype=torch.float64)
    Kd, Vd, Qd = K.cpu().double(), V.cpu().double(), Q.cpu().double()
    for h, spans in enumerate(idx[:, 0].tolist()):
        t = torch.cat([torch.arange(j * S, (j + 1) * S) for j in spans if 0 <= j < c] + [torch.arange(c * S, L)])
        z = Kd[h // 8][t] @ Qd[h, 0] / D ** 0.5
        exact[h], lse[h] = torch.softmax(z, 0) @ Vd[h // 8][t], torch.logsumexp(z, 0)
    assert float((O[:, 0].cpu().double() - exact).norm() / exact.norm()) <= 2.0 ** -22
    assert float((LSE[:, 0].cpu().double() - lse).norm() / lse.norm()) <= 2.0 ** -22


def test_armed_events_hold_the_kernel_of_a_short_decode_step():
    """Attached to the dispatch, they hold the kernel's own time, which is below what a call takes in a graph of such calls
    (6.2 of 6.5 us); recorded on the stream they held the dispatch gaps too (8.7 us)."""
    S, k = 64, 4
    L = S * 40
    Q, K, V = make(3250, 32, 4, L, 128, torch.bfloat16, Lq=1)
    idx = B.sl_span_search_decode(Q, K, None, S, k)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()                      # creates the handles
    kernel = []
    for _ in range(41):
        B.sl_span_attention_decode(Q, K, V, idx, S, prof=(ev[0].cuda_event, ev[1].cuda_event))
        torch.cuda.synchronize()
        kernel.append(ev[0].elapsed_time(ev[1]))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        B.sl_span_attention_decode(Q, K, V, idx, S)
    torch.cuda.synchronize()
    graph, outs = torch.cuda.CUDAGraph(), []
    with torch.cuda.graph(graph):
        for _ in range(100):
            outs.append(B.sl_span_attention_decode(Q, K, V, idx, S))
    calls = []
    for _ in range(5):
        ev[0].record()
        graph.replay()
        ev[1].record()
        torch.cuda.synchronize()
        calls.append(ev[0].elapsed_time(ev[1]) / 100)
    assert 0 < sorted(kernel)[20] <= 1.15 * sorted(calls)[2], (sorted(kernel), calls)


@pytest.mark.parametrize("Lq", [6143, 6145, 8200])    # 1536 workgroups, more of them; 4097 candidates at the last rows
@pytest.mark.parametrize("k", [4, 8])
def test_prefill_search_of_many_candidates_at_both_grid_sizes(Lq, k):
    """Few and many workgroups, which go different ways from 1025 and 2049 candidates on: the form that returns scores
    computes the same ones and carries no numbers in them, so the selections are equal."""
    L = 8200
    Q, K, V = make(3300 + Lq + k, 32, 4, L, 128, torch.bfloat16, Lq=Lq)
    idx = B.sl_span_search_prefill(Q, K, None, 2, k, q_pos0=L - Lq)
    two, _ = B.sl_span_search_prefill(Q, K, None, 2, k, q_pos0=L - Lq, want_scores=True)
    torch.cuda.synchronize()
    assert torch.equal(idx, two)


TILES = [
    # kind     Hq  Hkv L      Lq     S or w  A    k  blocks of the whole call's routed tiles and windows
    ("grid", 8, 1, 14001, 13000, 64, 64, 4, 2, 1),
    ("grid", 16, 1, 28011, 25000, 1024, 1024, 2, 2, 2),    # windows that merge
    ("gated", 8, 1, 14001, 13000, 64, 64, 4, 2, 1),
    ("gated", 16, 1, 28011, 25000, 1024, 1024, 2, 2, 2),   # windows that do not
    ("grid", 8, 1, 14001, 13000, 128, 64, 4, 2, 1),        # clipped spans
    ("gated", 8, 1, 14001, 13000, 128, 64, 4, 2, 1),       # whole spans that overlap
    ("anchor", 8, 1, 27003, 25000, 1088, 1, 2, 2, 2),
]


def end_block(Hq, Hkv, L, Lq, k, reach, tile_rows):
    """Tokens of an end block of the paper's geometry, in whose buckets rows share tiles."""
    x, span = Hq // Hkv * Lq * k / L, reach * math.ceil(math.sqrt(L - Lq + Lq // 2)) + 1
    best, E = math.sqrt(0.5 * tile_rows * span / x), 64
    while E < 4096 and E * 1.4142 < best:
        E *= 2
    while E > 64 and Hkv * (L / E + x * L / tile_rows) < 256:
        E //= 2
    return E


def column_blocks(kind, Hq, Hkv, L, Lq, S, A, k, reach=4):
    """Blocks of 32 columns that a wavefront of the routed and of the window kernel takes, and how far the sizes that decide it
    lie from the lines, as a factor."""
    tokens, slots = S if kind == "anchor" else A / 2, k
    if kind == "anchor":
        A = end_block(Hq, Hkv, L, Lq, k, reach, 256)
    else:                                        # slots of a row's list that it has candidates for, on average
        before = [i * i / A / 2 if i < k * A else k * (i - k * A / 2) for i in (L - Lq, L)]
        slots = (before[1] - before[0]) / Lq
    items = Hq * Lq * slots
    buckets = min(items, Hkv * max(1, L // A))
    routed = (items / (500 * buckets), (items / 256 + buckets / 2) / 1024)
    window = (Hq * Lq / (512 * 256), Hq * Lq * tokens / (2048 * 65536))
    return [(2 if min(f) >= 1 else 1, min(f) if min(f) >= 1 else 1 / min(f)) for f in (routed, window)]


def tile_call(kind, Q, K, V, idx, sc, S, A, q0):
    if kind == "anchor":
        return (B.sl_anchor_attention_prefill(Q, K, V, idx, sc, S, 3, 1, q_pos0=q0),)
    stride = 0 if A == S else A
    if kind == "gated":
        return (B.sl_span_attention_combined_prefill(Q, K, V, idx, sc, S, q_pos0=q0, span_stride=stride),)
    return B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0, span_stride=stride)


def tile_inputs(kind, Hq, Hkv, L, Lq, S, A, k):
    q0 = L - Lq
    Q, K, V = make(71, Hq, Hkv, L, 128, torch.bfloat16, scale=0.5, Lq=Lq)
    if kind == "anchor":
        idx, sc = B.sl_anchor_search_prefill(Q, K, k, S, q_pos0=q0, want_scores=True)
    else:
        idx, sc = B.sl_span_search_prefill(Q, K, None, A, k, q_pos0=q0, want_scores=True)
    return q0, Q, K, V, idx, torch.where(torch.isfinite(sc), sc, 0.0)


@pytest.mark.parametrize("kind,Hq,Hkv,L,Lq,S,A,k,routed,window", TILES)
def test_rows_are_alike_in_tiles_of_one_and_two_column_blocks(kind, Hq, Hkv, L, Lq, S, A, k, routed, window):
    """A long call takes tiles of two blocks of columns, its pieces of one: the same arithmetic for every row, whatever tile,
    wavefront (31 to 33, 63 to 65 rows) and kv rows at a time take it."""
    blocks = column_blocks(kind, Hq, Hkv, L, Lq, S, A, k)
    assert [b for b, _ in blocks] == [routed, window] and all(far >= 1.5 for b, far in blocks if b == 2)
    q0, Q, K, V, idx, sc = tile_inputs(kind, Hq, Hkv, L, Lq, S, A, k)
    whole = tile_call(kind, Q, K, V, idx, sc, S, A, q0)
    at = 0
    for n in (1, 31, 33, 65, 127, 129, 300, 1025):
        r0 = min(Lq - n, at)
        assert [b for b, _ in column_blocks(kind, Hq, Hkv, q0 + r0 + n, n, S, A, k)] == [1, 1]
        part = tile_call(kind, Q[:, r0:r0 + n].contiguous(), K[:, :q0 + r0 + n].contiguous(), V[:, :q0 + r0 + n].contiguous(),
                         idx[:, r0:r0 + n].contiguous(), sc[:, r0:r0 + n].contiguous(), S, A, q0 + r0)
        torch.cuda.synchronize()
        for w, p in zip(whole, part):
            assert torch.equal(w[:, r0:r0 + n], p), (kind, n, r0)
        at += Lq // 8


@pytest.mark.parametrize("rows", ["few", "many"])
@pytest.mark.parametrize("kind,Hq,Hkv,L,Lq,S,A,k", [t[:8] for t in TILES])
def test_queries_that_are_not_finite_reach_no_other_row(kind, Hq, Hkv, L, Lq, S, A, k, rows):
    """Row sums come from a product that mixes columns of a tile: a row whose scores are not numbers, or infinite, is NaN,
    and every other row is what it was."""
    q0, Q, K, V, idx, sc = tile_inputs(kind, Hq, Hkv, L, Lq, S, A, k)
    if rows == "few":
        q0, Q, idx, sc = q0 + Lq - 200, Q[:, -200:].contiguous(), idx[:, -200:].contiguous(), sc[:, -200:].contiguous()
    clean = tile_call(kind, Q, K, V, idx, sc, S, A, q0)
    spoilt, bad = Q.clone(), torch.zeros(Q.shape[:2], dtype=torch.bool, device=DEV)
    for h, r, x in ((0, 3, math.nan), (Hq - 1, Q.shape[1] // 2, math.nan), (1, 17, math.inf), (2, Q.shape[1] - 1, -math.inf)):
        spoilt[h, r, 5] = x
        bad[h, r] = True
    got = tile_call(kind, spoilt, K, V, idx, sc, S, A, q0)
    torch.cuda.synchronize()
    assert bool(torch.isnan(got[0][bad]).all())
    for c, g in zip(clean, got):
        assert torch.equal(c[~bad], g[~bad])


@pytest.mark.parametrize("Hq,Lq,k,b,run", [(16, 1000, 1, 2, 64), (32, 8000, 3, 20, 128)])   # one block of columns, two
def test_anchor_wavefronts_pass_over_what_none_of_their_rows_attends(Hq, Lq, k, b, run):
    """Rows of one end block in runs of two wavefronts, one's span ends 140 or 180 tokens behind the other's: the tile's last kv rows, one of whose V
    is not a number, are attended by every other run alone."""
    L, w = 9000, 255
    t0, t1 = (5140, 5280) if Lq == 1000 else (520, 700)
    blocks = column_blocks("anchor", Hq, Hq, L, Lq, w, 1, k, reach=b)[0][0]
    E = end_block(Hq, Hq, L, Lq, k, b, 128 * blocks)
    assert blocks == (1 if Lq == 1000 else 2) and t0 // E == t1 // E
    Q, K, V = make(33, Hq, Hq, L, 128, torch.bfloat16, scale=0.5, Lq=Lq)
    late = torch.arange(Lq, device=DEV) // run % 2 == 1
    an = torch.full((Hq, Lq, k), -1, dtype=torch.int32, device=DEV)
    an[:, :, 0] = torch.where(late, t1, t0)
    sc = torch.zeros((Hq, Lq, k), dtype=torch.float32, device=DEV)
    spoilt = V.clone()
    spoilt[:, t1 - 1, 7] = math.nan
    clean, got = (B.sl_anchor_attention_prefill(Q, K, v, an, sc, w, b, 0, q_pos0=L - Lq) for v in (V, spoilt))
    torch.cuda.synchronize()
    assert bool(torch.isnan(got[:, late, 7]).all())
    assert torch.equal(got[:, ~late], clean[:, ~late])


def test_anchor_wavefronts_pass_over_what_lies_between_their_rows_spans():
    """Rows of a wavefront whose spans lie apart, with 64 kv rows between them that none attends, one of whose V is not a number."""
    H, L, Lq, w, t0, t1 = 16, 9000, 1000, 255, 5130, 5370
    E = end_block(H, H, L, Lq, 1, 1, 128)
    assert t0 // E == t1 // E and t1 - math.ceil(math.sqrt(L)) > 5248 and column_blocks("anchor", H, H, L, Lq, w, 1, 1, reach=1)[0][0] == 1
    Q, K, V = make(35, H, H, L, 128, torch.bfloat16, scale=0.5, Lq=Lq)
    an = torch.where(torch.arange(Lq, device=DEV) % 2 == 1, t1, t0).to(torch.int32).expand(H, Lq)[:, :, None].contiguous()
    sc = torch.zeros((H, Lq, 1), dtype=torch.float32, device=DEV)
    spoilt = V.clone()
    spoilt[:, 5210] = math.nan
    clean, got = (B.sl_anchor_attention_prefill(Q, K, v, an, sc, w, 1, 0, q_pos0=L - Lq) for v in (V, spoilt))
    torch.cuda.synchronize()
    assert torch.equal(got, clean)


def lse_with_rounded_weights(Q, K, idx, S, A, q0, rows):
    """(lse as bf16-weight tiles have it, lse) in 64 bits, [Hq, rows].  A partial (a span, the window) goes 64 keys at a time;
    its weights are rounded to bf16 against a bound, which the first 64 keys' maximum sets and a maximum moves that exceeds it
    by more than 8 (log2 units)."""
    Hq, _, D = Q.shape
    G, k, n = Hq // K.shape[0], idx.shape[2], rows.numel()
    kv = torch.arange(Hq, device=DEV)[:, None] // G
    q = Q[:, rows].double() / (math.sqrt(D) * math.log(2))
    pos, spans = q0 + rows, idx[:, rows].long()
    ok = (spans >= 0) & (spans < (pos // A)[None, :, None])
    parts, exact = [], []
    for s in range(k + 1):
        if s < k:
            end = (spans[:, :, s] + 1) * A
            lo = start = (end - S).clamp(min=0)
            for t in range(k if A < S else 0):                    # a token of the union counts once
                lo = torch.where(ok[:, :, t] & (spans[:, :, t] < spans[:, :, s]), torch.maximum(lo, (spans[:, :, t] + 1) * A), lo)
            use, steps = ok[:, :, s], S // 64
        else:
            end = (pos + 1).expand(Hq, n)
            lo = start = (pos // A * A).expand(Hq, n)
            use, steps = torch.ones_like(ok[:, :, 0]), A // 64
        m = torch.full((Hq, n), -math.inf, dtype=torch.float64, device=DEV)
        l, total = torch.zeros_like(m), torch.zeros_like(m)
        for c in range(steps):
            at = start[:, :, None] + 64 * c + torch.arange(64, device=DEV)
            keys = K[kv[:, :, None], at.clamp(0, K.shape[1] - 1)].double()
            z = (keys @ q[:, :, :, None])[..., 0]
            z = z.masked_fill((at < lo[:, :, None]) | (at >= end[:, :, None]), -math.inf)
            top = z.amax(dim=2)
            to = torch.where(top > m + 8, top, m)
            to0 = torch.where(torch.isinf(to), 0.0, to)
            p = torch.exp2(z - to0[:, :, None])
            l = l * torch.exp2(m - to0) + p.float().bfloat16().double().sum(dim=2)
            total = total * torch.exp2(m - to0) + p.sum(dim=2)
            m = to
        gone = ~use
        parts.append(((m + l.log2()) * math.log(2)).masked_fill(gone, -math.inf))
        exact.append(((m + total.log2()) * math.log(2)).masked_fill(gone, -math.inf))
    return torch.logsumexp(torch.stack(parts), dim=0), torch.logsumexp(torch.stack(exact), dim=0)


@pytest.mark.parametrize("S,A,k", [(64, 64, 8), (64, 64, 16), (128, 128, 8), (128, 64, 8), (192, 64, 8)])
@pytest.mark.parametrize("Lq", [8200, 300])          # tiles of two blocks of columns, of one
@pytest.mark.parametrize("std", [1.0, 1.5])
def test_heaviest_weight_of_a_span_is_not_rounded(S, A, k, Lq, std):
    """The error of lse is that of weights rounded to bf16 with the heaviest of a span's first 64 keys a power of two, and no
    more.  Scores in 32 bits turn the rounding of one weight in a thousand, which moves the root mean square over thousands of
    rows by far less than 3 %; a bound from the first 32 keys alone makes it 12 % larger at spans of 64 and unit variance, 4 % at
    128, and more with steeper scores."""
    L, q0 = 9000, 9000 - Lq
    assert column_blocks("grid", 8, 1, L, Lq, S, A, k)[0][0] == (2 if Lq > 300 else 1)
    Q, K, V = make(90 + S + A, 8, 1, L, 128, torch.bfloat16, scale=std, Lq=Lq)
    idx = B.sl_span_search_prefill(Q, K, None, A, k, q_pos0=q0)
    _, LSE = B.sl_span_attention_prefill(Q, K, V, idx, S, q_pos0=q0, span_stride=0 if A == S else A)
    torch.cuda.synchronize()
    rows = torch.arange(0, Lq, max(1, Lq // 300), device=DEV)
    want, exact = lse_with_rounded_weights(Q, K, idx, S, A, q0, rows)
    seen = (LSE[:, rows].double() - exact).pow(2).mean().sqrt()
    allowed = (want - exact).pow(2).mean().sqrt()
    assert float(seen) <= 1.03 * float(allowed), (float(seen), float(allowed))


@pytest.mark.parametrize("Hq,Hkv,L,D,S,A,k,form,q_pos0,Lq", [
    (8, 2, 4000, 128, 33, 33, 8, "joint", 0, 4000),          # a span is two steps, the second of one token
    (8, 2, 5000, 128, 31, 31, 8, "gated", 0, 5000),          # one step, and no other
    (8, 2, 6000, 128, 97, 50, 8, "joint", 0, 6000),          # overlapping spans, a last step of one token
    (32, 4, 6000, 128, 129, 129, 8, "joint", 5000, 1000),    # many tiles: stages of 32 tokens
    (8, 8, 4488, 128, 838, 838, 2, "gated", 4412, 76),       # few: of 64
    (4, 1, 3000, 128, 641, 641, 4, "joint", 2700, 300),
    (4, 1, 3000, 128, 703, 400, 4, "joint", 2700, 300),
    (8, 2, 5000, 64, 65, 65, 8, "joint", 0, 5000),
    (8, 2, 5000, 64, 97, 40, 8, "joint", 0, 5000),
])
def test_steps_and_stages_of_any_span_length(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq):
    """Spans that end with or one token behind a step of 32 kv rows or a stage, stages of both lengths, on
    test_any_span_length_on_the_matrix_cores's terms."""
    test_any_span_length_on_the_matrix_cores(Hq, Hkv, L, D, S, A, k, form, q_pos0, Lq)
