"""GPU parity of the LM-head projection fused with the candidate sets (ubt_lm_head_topk)
against the fp64 oracle, through the C ABI.

* Integer-valued hidden states and head rows: every logit is an exact integer in fp32,
  whatever the accumulation order, so ids and logits must match bit for bit, and the many
  equal logits test the tie order (id asc) across tiles, waves and workgroups.  With the
  binding's full workspace, calls of up to 16 rows run the kernel that splits d over a
  workgroup's waves where it takes d (every slice width) and all others run the matrix
  product; with a workspace of the plain query's size, calls of several row groups run the
  split kernel or the one that does not split d.
* Gaussian operands at the drafting block of the paper's latency breakdown (16 rows of a
  2560-wide hidden state against a 151,936-token head), at d = 4096, and at small and
  ragged shapes (M not a multiple of 16, V not a multiple of 16, d/32 odd): logits within
  the derived fp32 accumulation bound, the candidate order valid under it.
* Degenerate cases: h = 0 (every logit 0), K = V, K = 1, one row; reuse of a workspace
  across calls of different shapes and kernels."""
from __future__ import annotations

import math

import numpy as np
import pytest

import parity
import synth

pytestmark = pytest.mark.gpu


def _run(h_bits, w_bits, K, workspace=None):
    import torch

    import paper_2609_39972_amd as ubt

    h = ubt.bf16_tensor_from_bits(h_bits)
    w = ubt.bf16_tensor_from_bits(w_bits)
    out = ubt.lm_head_topk(h, w, K, workspace=workspace)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items() if v is not None}


def _int_bits(M, d, V, seed, lo=-8, hi=8):
    rng = np.random.default_rng(seed)
    h = rng.integers(lo, hi + 1, size=(M, d)).astype(np.float64)
    w = rng.integers(lo, hi + 1, size=(V, d)).astype(np.float64)
    return synth.round_bf16_bits(h), synth.round_bf16_bits(w)


@pytest.mark.parametrize("M,d,V,K", [
    # d not a multiple of 512: one wave per tile over the whole of d
    (1, 32, 64, 1), (5, 96, 1000, 8), (16, 256, 4099, 64), (17, 64, 2500, 16), (33, 128, 777, 64),
    # d a multiple of 512: the eight waves of a workgroup split d (every slice width built)
    (3, 2560, 3000, 64), (2, 1024, 3001, 64), (16, 1536, 4099, 64), (17, 2048, 1500, 16), (5, 3072, 999, 8),
    (5, 3584, 2000, 8), (1, 4096, 130, 64), (1, 5120, 777, 64), (20, 2560, 70001, 64),
])
def test_lm_head_integer_inputs_exact(M, d, V, K):
    print(f"lm_head exact M={M} d={d} V={V} K={K}", flush=True)
    hb, wb = _int_bits(M, d, V, seed=M * 1000 + d + V)
    g = _run(hb, wb, K)
    parity.check_lm_head(g, hb, wb, K, exact=True)


def test_lm_head_ties_in_many_workgroups():
    """Heads with only a few distinct rows: most logits tie, across every workgroup."""
    print("lm_head ties", flush=True)
    rng = np.random.default_rng(7)
    base = rng.integers(-4, 5, size=(3, 64)).astype(np.float64)
    wb = synth.round_bf16_bits(base[rng.integers(0, 3, size=20011)])
    hb = synth.round_bf16_bits(rng.integers(-4, 5, size=(9, 64)).astype(np.float64))
    parity.check_lm_head(_run(hb, wb, 64), hb, wb, 64, exact=True)


@pytest.mark.parametrize("M,d,V,K,seed", [
    (15, 2560, 151936, 64, 1),   # the drafting block of the paper's latency breakdown
    (16, 4096, 151936, 64, 2),
    (1, 64, 1000, 8, 3),
    (17, 96, 5003, 16, 4),
    (40, 256, 20000, 64, 5),
    (3, 2560, 32000, 1, 6),
])
def test_lm_head_gaussian(M, d, V, K, seed):
    print(f"lm_head gaussian M={M} d={d} V={V} K={K} seed={seed}", flush=True)
    x = synth.lm_head_inputs(seed, M, d, V)
    counts = parity.check_lm_head(_run(x["h"], x["w"], K), x["h"], x["w"], K)
    parity.record(f"lm_head M={M} d={d} V={V} K={K}", {"exact": counts["exact"], "excused": counts["excused"]})


def test_lm_head_zero_hidden_state():
    """h = 0: every logit is 0, so C = ids 0..K-1 and LSE = ln V."""
    print("lm_head zero h", flush=True)
    V, d = 70001, 128
    x = synth.lm_head_inputs(8, 1, d, V)
    hb = np.zeros((4, d), np.uint16)
    g = _run(hb, x["w"], 64)
    np.testing.assert_array_equal(g["cand_ids"], np.tile(np.arange(64), (4, 1)))
    np.testing.assert_array_equal(g["cand_logit"], 0.0)
    np.testing.assert_allclose(g["lse"], math.log(V), rtol=1e-6)
    np.testing.assert_allclose(g["cand_logprob"], -math.log(V), rtol=1e-6)


def test_lm_head_k_equals_v():
    print("lm_head K = V", flush=True)
    x = synth.lm_head_inputs(9, 6, 64, 64)
    g = _run(x["h"], x["w"], 64)
    parity.check_lm_head(g, x["h"], x["w"], 64)
    assert all(sorted(r.tolist()) == list(range(64)) for r in g["cand_ids"])


def test_lm_head_workspace_reuse():
    """One workspace (sized for the larger call) serves calls of different shapes in a
    row; nothing carries over between them."""
    import paper_2609_39972_amd as ubt

    print("lm_head workspace reuse", flush=True)
    ws = ubt.lm_head_workspace(40, 128, 50000, 64)
    a = synth.lm_head_inputs(10, 40, 128, 50000)
    b = synth.lm_head_inputs(11, 7, 128, 3001)
    for x, K in ((a, 64), (b, 8), (a, 64)):
        parity.check_lm_head(_run(x["h"], x["w"], K, workspace=ws), x["h"], x["w"], K)


def test_lm_head_workspace_reuse_across_shapes():
    """One workspace serves calls with different numbers of row groups, hidden sizes and
    kernels in any order: nothing in it is read before the call writes it."""
    import paper_2609_39972_amd as ubt

    print("lm_head workspace reuse across shapes", flush=True)
    cases = [(40, 2560, 30011, 64), (5, 2560, 9000, 8), (17, 1024, 20000, 16), (3, 96, 3000, 4), (40, 2560, 30011, 64)]
    n = max(ubt.lib().ubt_lm_head_topk_workspace_bytes(M, d, V, K) for M, d, V, K in cases)
    import torch
    ws = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")  # stale bytes must not matter
    for i, (M, d, V, K) in enumerate(cases):
        x = synth.lm_head_inputs(20 + i, M, d, V)
        parity.check_lm_head(_run(x["h"], x["w"], K, workspace=ws), x["h"], x["w"], K)


@pytest.mark.parametrize("M,d,V,K", [
    # One row block of every height (32 rows per step), d / 32 odd and even, one k stage and many
    (32, 32, 700, 8), (48, 96, 4099, 64), (65, 128, 2000, 16), (128, 224, 4097, 10), (130, 64, 5003, 64),
    (160, 1024, 2049, 64),
    # Two to four row blocks (the last rows of the last past M), several products per call
    (161, 320, 1000, 8), (193, 96, 3333, 4), (257, 64, 3000, 8), (320, 544, 3000, 8), (321, 96, 1500, 16),
    (480, 160, 70001, 8), (512, 1120, 1000, 64), (530, 64, 5000, 64), (1030, 32, 300, 8),
    # One stage per partial sum, several, and a last one that is shorter
    (33, 512, 2000, 8), (33, 576, 2000, 8), (33, 1088, 2000, 8), (33, 2880, 2000, 8),
    # Ranges of several tiles per workgroup, the last tile of one to four 64-row passes
    (17, 64, 151936, 8), (40, 64, 100003, 16), (20, 32, 262145, 4),
    # Up to 16 rows where d is no multiple of 512
    (1, 96, 5000, 8), (15, 2880, 3001, 64), (16, 160, 40001, 16),
])
def test_lm_head_product_integer_inputs_exact(M, d, V, K):
    """The matrix product (more than 16 rows, or d no multiple of 512): integer-valued
    inputs, so every logit is exact in fp32 and ids, ties included, must match bit for bit.
    The workspace starts out filled with a pattern: nothing in it is read unwritten."""
    import paper_2609_39972_amd as ubt

    print(f"lm_head product M={M} d={d} V={V} K={K}", flush=True)
    hb, wb = _int_bits(M, d, V, seed=M * 1000 + d + V, lo=-3, hi=3)
    ws = ubt.lm_head_workspace(M, d, V, K)
    assert ws.numel() >= min(M, 512) * V * 4  # room for the logits: the product runs
    ws.fill_(0x7F)  # as fp32: 3.4e38, above every logit
    parity.check_lm_head(_run(hb, wb, K, workspace=ws), hb, wb, K, exact=True)


@pytest.mark.parametrize("K", [1, 64])
def test_lm_head_product_all_logits_tied(K):
    """h = 0 in some rows: all of the row's logits tie, far more than the select kernel ranks
    in LDS; the lowest ids win."""
    print(f"lm_head product ties K={K}", flush=True)
    hb, wb = _int_bits(24, 64, 30011, seed=5)
    hb[::2] = 0
    parity.check_lm_head(_run(hb, wb, K), hb, wb, K, exact=True)


def test_lm_head_product_and_row_groups_agree():
    """A workspace of the plain query's size (smaller than the product needs here) keeps a call
    with many rows on the row-group kernels; both routes give the same ids and values on
    exact inputs."""
    import torch

    import paper_2609_39972_amd as ubt

    print("lm_head product against row groups", flush=True)
    hb, wb = _int_bits(40, 512, 30011, seed=6)
    small = torch.empty(ubt.lib().ubt_lm_head_topk_workspace_bytes(40, 512, 30011, 16), dtype=torch.uint8, device="cuda")
    assert small.numel() < ubt.lm_head_workspace(40, 512, 30011, 16).numel()
    a, b = _run(hb, wb, 16, workspace=small), _run(hb, wb, 16)
    for k in ("cand_ids", "cand_logit"):
        np.testing.assert_array_equal(a[k], b[k])
    np.testing.assert_allclose(a["lse"], b["lse"], rtol=1e-6)


@pytest.mark.parametrize("M,d,V,K", [
    # d split over the waves, two and three row groups (the last of 1, 4 and 16 rows)
    (17, 2048, 30000, 16), (20, 2560, 70001, 64), (48, 1024, 20000, 8),
    # the kernel that does not split d: up to 16 rows and several groups, d / 32 odd and even, d = 512
    (5, 96, 40001, 8), (16, 2880, 40001, 8), (33, 96, 60001, 16), (17, 2880, 20001, 8), (33, 512, 40000, 8),
])
def test_lm_head_row_groups_integer_inputs_exact(M, d, V, K):
    """A workspace of the plain size, too small for the product, keeps the call on the kernels
    that read the head once per 16 rows."""
    import paper_2609_39972_amd as ubt

    print(f"lm_head row groups M={M} d={d} V={V} K={K}", flush=True)
    hb, wb = _int_bits(M, d, V, seed=M * 1000 + d + V, lo=-3, hi=3)
    ws = ubt.lm_head_workspace(M, d, V, K, full=False)
    assert ws.numel() < min(M, 512) * V * 4  # no room for the logits
    ws.fill_(0x7F)
    parity.check_lm_head(_run(hb, wb, K, workspace=ws), hb, wb, K, exact=True)


@pytest.mark.parametrize("M,d,V,K", [
    # fewer than K thread pairs of the select kernel hold a group of 64 columns, in one range or in
    # many: fewer columns than threads, one column per thread, the last such length and the first past it
    (5, 96, 64, 64), (5, 96, 300, 64), (17, 96, 500, 33), (17, 64, 1500, 64), (200, 64, 1500, 64), (200, 96, 4097, 64),
    (480, 32, 8128, 64), (480, 32, 8257, 64), (300, 64, 5000, 64), (480, 64, 1000, 17),
    # the product where both it and the row groups take d
    (160, 1024, 2800, 64),
])
def test_lm_head_product_few_columns_exact(M, d, V, K):
    """Exact logits, with every logit of some rows tied (the lowest ids win)."""
    import paper_2609_39972_amd as ubt

    print(f"lm_head product few columns M={M} d={d} V={V} K={K}", flush=True)
    hb, wb = _int_bits(M, d, V, seed=M + d + V, lo=-3, hi=3)
    hb[::5] = 0
    ws = ubt.lm_head_workspace(M, d, V, K)
    ws.fill_(0x7F)
    parity.check_lm_head(_run(hb, wb, K, workspace=ws), hb, wb, K, exact=True)


@pytest.mark.parametrize("M,V", [(17, 1500), (480, 4000)])
def test_lm_head_few_columns_take_little_longer_at_large_k(M, V):
    """K = 64 against K = 8, d = 2880, where K = 64 thread pairs do not each hold a group: without a
    bound the select kernel ranked or selected among every element (17 x 1,500: 91.9 us against 28.4;
    480 x 4,000: 82.2 against 45.5; with one 37.4 and 51.3)."""
    import torch

    import paper_2609_39972_amd as ubt
    from gpu_util import best_us

    h, w = torch.randn(M, 2880, device="cuda").bfloat16(), torch.randn(V, 2880, device="cuda").bfloat16()

    def us(K):
        ws = ubt.lm_head_workspace(M, 2880, V, K)
        out = ubt.lm_head_topk(h, w, K, workspace=ws)
        return best_us(lambda: ubt.lm_head_topk(h, w, K, out=out, workspace=ws))

    few, many = us(8), us(64)
    print(f"M={M} V={V}: K = 8 {few:.1f} us, K = 64 {many:.1f} us", flush=True)
    assert many < 1.6 * few
