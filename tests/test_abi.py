"""The C ABI of libubt.so on the host: exported symbols, status strings and
argument validation, which returns an error before any device work (so
these run without a GPU; the pointers passed are never dereferenced)."""
from __future__ import annotations

import ctypes
import re
import subprocess

import pytest

import paper_2609_39972_amd as ubt

FAKE = ctypes.c_void_p(0x10000)  # never dereferenced: every call below fails validation first


def _declared() -> set:
    hdr = open(f"{ubt.PKG}/../include/ubt.h").read()
    return set(re.findall(r"\b(ubt_[a-z_]+)\s*\(", hdr))


def test_library_exports_every_declared_symbol():
    L = ubt.lib()
    declared = _declared()
    assert declared == set(ubt.EXPORTS)
    nm = subprocess.run(["nm", "-D", "--defined-only", ubt.LIB_PATH], capture_output=True, text=True, check=True)
    exported = set(re.findall(r" T (ubt_\w+)", nm.stdout))
    assert declared <= exported
    for name in declared:
        assert hasattr(L, name)


def test_version_and_status_strings():
    L = ubt.lib()
    assert L.ubt_abi_version() == 1
    for code, name in ubt.STATUS.items():
        assert L.ubt_status_str(code).decode() == name
    assert L.ubt_status_str(99).decode() == "UBT_ERR_UNKNOWN"


def _topk(**kw):
    a = dict(logits=FAKE, dt=1, B=2, gamma=3, V=1000, sb=3000, si=1000, K=8, ids=FAKE, val=FAKE, lp=None, lse=None)
    a.update(kw)
    return ubt.lib().ubt_topk(a["logits"], a["dt"], a["B"], a["gamma"], a["V"], a["sb"], a["si"], a["K"], a["ids"],
                              a["val"], a["lp"], a["lse"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(logits=None), 1), (dict(ids=None), 1), (dict(val=None), 1),
    (dict(dt=5), 3),
    (dict(B=0), 2), (dict(gamma=0), 2), (dict(gamma=65), 2), (dict(K=0), 2), (dict(K=65), 2), (dict(V=7), 2),
    (dict(si=999), 2), (dict(sb=2999), 2), (dict(V=2 ** 31, si=2 ** 31, sb=3 * 2 ** 31), 2),
])
def test_topk_validation(kw, code):
    assert _topk(**kw) == code


def _bigram(alpha=None, lam=None, **kw):
    g = kw.pop("gamma", 3)
    a = (ctypes.c_float * 64)(*([1.0] * 64)) if alpha is None else alpha
    l_ = (ctypes.c_float * 64)(*([1.0] * 64)) if lam is None else lam
    args = dict(phi=FAKE, psi=FAKE, gate=FAKE, dt=1, V=1000, r=64, anchor=FAKE, ids=FAKE, logit=FAKE, B=2, K=8,
                delta=None, logq=FAKE)
    args.update(kw)
    return ubt.lib().ubt_bigram_scores(args["phi"], args["psi"], args["gate"], args["dt"], args["V"], args["r"],
                                       args["anchor"], args["ids"], args["logit"], a, l_, args["B"], g, args["K"],
                                       args["delta"], args["logq"], None)


def _arr(vals):
    return (ctypes.c_float * len(vals))(*vals)


@pytest.mark.parametrize("kw,code", [
    (dict(phi=None), 1), (dict(gate=None), 1), (dict(anchor=None), 1), (dict(logq=None), 1),
    (dict(dt=9), 3), (dict(r=8), 2), (dict(r=72), 2), (dict(r=528), 2), (dict(K=65), 2), (dict(gamma=65), 2),
    (dict(V=5), 2), (dict(B=0), 2),
    (dict(alpha=_arr([1.0, 0.0, 1.0])), 3), (dict(lam=_arr([1.0, 1.0, -2.0])), 3),
    (dict(alpha=_arr([1.0, float("inf"), 1.0])), 3), (dict(lam=_arr([float("nan"), 1.0, 1.0])), 3),
    (dict(phi=ctypes.c_void_p(0x10002)), 4),
])
def test_bigram_validation(kw, code):
    assert _bigram(**kw) == code


def _tree(dbg=None, **kw):
    a = dict(anchor=FAKE, ids=FAKE, logq=FAKE, B=2, gamma=15, K=8, W=12, budget=64, zeta=0.0, nn=FAKE, tok=FAKE,
             par=FAKE, dep=FAKE, cr=FAKE, sc=FAKE, mask=None)
    a.update(kw)
    return ubt.lib().ubt_build_tree(a["anchor"], a["ids"], a["logq"], a["B"], a["gamma"], a["K"], a["W"],
                                    a["budget"], a["zeta"], a["nn"], a["tok"], a["par"], a["dep"], a["cr"], a["sc"],
                                    a["mask"], dbg, None)


@pytest.mark.parametrize("kw,code", [
    (dict(anchor=None), 1), (dict(logq=None), 1), (dict(nn=None), 1), (dict(sc=None), 1),
    (dict(B=0), 2), (dict(gamma=0), 2), (dict(gamma=65), 2), (dict(K=65), 2), (dict(W=0), 2), (dict(W=256), 2),
    (dict(budget=0), 2), (dict(budget=256), 2),
    (dict(W=65, K=64), 4), (dict(gamma=64, W=65, K=4), 4),
    (dict(zeta=0.5), 3), (dict(zeta=float("-inf")), 3), (dict(zeta=float("nan")), 3),
])
def test_build_tree_validation(kw, code):
    assert _tree(**kw) == code


def test_build_tree_incomplete_debug_struct():
    s = ubt._Supertree(FAKE, None, FAKE, FAKE)
    assert _tree(dbg=ctypes.byref(s)) == 1


def _draft(alpha=None, lam=None, **kw):
    a_ = (ctypes.c_float * 64)(*([1.0] * 64)) if alpha is None else alpha
    l_ = (ctypes.c_float * 64)(*([1.0] * 64)) if lam is None else lam
    a = dict(phi=FAKE, psi=FAKE, gate=FAKE, dt=1, V=1000, r=64, anchor=FAKE, ids=FAKE, logit=FAKE, B=2, gamma=3,
             K=8, W=4, budget=10, zeta=0.0, logq=FAKE, nn=FAKE, tok=FAKE, par=FAKE, dep=FAKE, cr=FAKE, sc=FAKE,
             mask=None)
    a.update(kw)
    return ubt.lib().ubt_draft_tree(a["phi"], a["psi"], a["gate"], a["dt"], a["V"], a["r"], a["anchor"], a["ids"],
                                    a["logit"], a_, l_, a["B"], a["gamma"], a["K"], a["W"], a["budget"], a["zeta"],
                                    a["logq"], a["nn"], a["tok"], a["par"], a["dep"], a["cr"], a["sc"], a["mask"],
                                    None)


@pytest.mark.parametrize("kw,code", [
    (dict(phi=None), 1), (dict(logit=None), 1), (dict(logq=None), 1), (dict(nn=None), 1), (dict(sc=None), 1),
    (dict(dt=9), 3), (dict(r=8), 2), (dict(K=65), 2), (dict(gamma=65), 2), (dict(V=5), 2), (dict(B=0), 2),
    (dict(W=0), 2), (dict(budget=256), 2), (dict(W=65, K=64), 4), (dict(gamma=64, W=65, K=4), 4),
    (dict(alpha=_arr([1.0, 0.0, 1.0])), 3), (dict(lam=_arr([1.0, 1.0, float("nan")])), 3),
    (dict(zeta=0.5), 3), (dict(zeta=float("nan")), 3), (dict(gate=ctypes.c_void_p(0x10008)), 4),
])
def test_draft_tree_validation(kw, code):
    """The one-call selector + search checks the union of the two calls' arguments."""
    assert _draft(**kw) == code


@pytest.mark.parametrize("args,code", [
    ((None, FAKE, 2, 65, FAKE), 1), ((FAKE, None, 2, 65, FAKE), 1), ((FAKE, FAKE, 2, 65, None), 1),
    ((FAKE, FAKE, 0, 65, FAKE), 2), ((FAKE, FAKE, 2, 0, FAKE), 2), ((FAKE, FAKE, 2, 257, FAKE), 2),
])
def test_tree_mask_validation(args, code):
    assert ubt.lib().ubt_tree_mask(*args, None) == code


def test_binding_refuses_host_tensors():
    import torch

    with pytest.raises(ValueError):
        ubt.topk(torch.zeros(1, 1, 16, dtype=torch.bfloat16), 4)


def _attn(**kw):
    a = dict(q=FAKE, kc=FAKE, vc=FAKE, plen=FAKE, Pmax=128, kt=FAKE, vt=FAKE, mask=FAKE, nn=FAKE, B=2, N=65, H=32,
             Hkv=8, D=128, scale=0.088, out=FAKE, odt=1, lse=None)
    a.update(kw)
    return ubt.lib().ubt_tree_attention(a["q"], a["kc"], a["vc"], a["plen"], a["Pmax"], a["kt"], a["vt"], a["mask"],
                                        a["nn"], a["B"], a["N"], a["H"], a["Hkv"], a["D"], a["scale"], a["out"],
                                        a["odt"], a["lse"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), 1), (dict(kt=None), 1), (dict(vt=None), 1), (dict(mask=None), 1), (dict(nn=None), 1),
    (dict(out=None), 1), (dict(plen=None), 1), (dict(kc=None), 1), (dict(vc=None), 1),
    (dict(B=0), 2), (dict(N=0), 2), (dict(N=257), 2), (dict(H=0), 2), (dict(Hkv=0), 2), (dict(H=30), 2),
    (dict(Pmax=-1), 2), (dict(Pmax=2 ** 31), 2),
    (dict(D=96), 4), (dict(D=256), 4), (dict(q=ctypes.c_void_p(0x10008)), 4), (dict(kc=ctypes.c_void_p(0x10004)), 4),
    (dict(odt=7), 3), (dict(scale=0.0), 3), (dict(scale=float("inf")), 3), (dict(scale=-1.0), 3),
])
def test_tree_attention_validation(kw, code):
    assert _attn(**kw) == code


def test_tree_attention_without_context_needs_no_cache():
    """P_max = 0 takes NULL caches; the call then fails only on what is still wrong."""
    assert _attn(Pmax=0, kc=None, vc=None, N=0) == 2


@pytest.mark.parametrize("args,code", [
    ((None, FAKE, FAKE, FAKE, 2, 65, FAKE, FAKE, FAKE), 1), ((FAKE, FAKE, FAKE, None, 2, 65, FAKE, FAKE, FAKE), 1),
    ((FAKE, FAKE, FAKE, FAKE, 2, 65, FAKE, FAKE, None), 1),
    ((FAKE, FAKE, FAKE, FAKE, 0, 65, FAKE, FAKE, FAKE), 2), ((FAKE, FAKE, FAKE, FAKE, 2, 257, FAKE, FAKE, FAKE), 2),
])
def test_verify_accept_validation(args, code):
    assert ubt.lib().ubt_verify_accept(*args, None) == code


@pytest.mark.parametrize("kw,code", [
    (dict(kt=None), 1), (dict(kc=None), 1), (dict(plen=None), 1), (dict(nodes=None), 1),
    (dict(B=0), 2), (dict(N=300), 2), (dict(Hkv=0), 2), (dict(Pmax=0), 2), (dict(D=32), 4),
    (dict(kc=ctypes.c_void_p(0x10002)), 4),
])
def test_commit_kv_validation(kw, code):
    a = dict(kt=FAKE, vt=FAKE, nodes=FAKE, alen=FAKE, plen=FAKE, kc=FAKE, vc=FAKE, B=2, N=65, Hkv=8, D=128, Pmax=64)
    a.update(kw)
    assert ubt.lib().ubt_commit_kv(a["kt"], a["vt"], a["nodes"], a["alen"], a["plen"], a["kc"], a["vc"], a["B"],
                                   a["N"], a["Hkv"], a["D"], a["Pmax"], None) == code


def _kl(**kw):
    g = kw.pop("gamma", 3)
    a = (ctypes.c_float * 64)(*([1.0] * 64))
    args = dict(logits=FAKE, dt=1, B=2, gamma=g, V=1000, sb=3000, si=1000, lse=FAKE, ids=FAKE, cl=FAKE, K=8, z=FAKE,
                tsb=3000, tsi=1000, y=FAKE, anchor=FAKE, phi=FAKE, psi=FAKE, gate=FAKE, fdt=1, r=64, alpha=a, lam=a,
                T=1.0, beta=0.1, loss=FAKE, kl=None, ce=None, gs=None, grad=None)
    args.update(kw)
    v = list(args.values())
    return ubt.lib().ubt_tree_kl_loss(*v, None)


@pytest.mark.parametrize("kw,code", [
    (dict(logits=None), 1), (dict(lse=None), 1), (dict(z=None), 1), (dict(y=None), 1), (dict(loss=None), 1),
    (dict(ids=None), 1), (dict(phi=None), 1), (dict(anchor=None), 1),
    (dict(dt=4), 3), (dict(fdt=4), 3), (dict(T=-0.5), 3), (dict(T=float("nan")), 3), (dict(beta=-1.0), 3),
    (dict(B=0), 2), (dict(K=65), 2), (dict(r=24), 2), (dict(si=999), 2), (dict(tsi=999), 2), (dict(tsb=2999), 2),
    (dict(grad=ctypes.c_void_p(0x10004)), 4), (dict(gate=ctypes.c_void_p(0x10008)), 4),
])
def test_tree_kl_loss_validation(kw, code):
    assert _kl(**kw) == code


def _step_ws_expected(B, gamma, V, K, es):
    """Workspace of the one-launch step: an error word, then 256-byte aligned regions
    for the row counters, the chunk ids and logits (C K each per row) and the chunk LSEs,
    with C = min(2, 64 // K, tiles per row) chunks of whole tiles (64 lanes x 64 bytes)."""
    al = lambda n: (n + 255) // 256 * 256
    tile = 64 * 64 // es
    tiles = -(-V // tile)
    c = min(2, max(1, 64 // K), tiles)
    length = -(-tiles // c) * tile
    C = -(-V // length)
    rows = B * gamma
    return 256 + al(rows * 4) + 2 * al(rows * C * K * 4) + al(rows * C * 4)


@pytest.mark.parametrize("B,gamma,V,K,dt", [
    (32, 15, 151936, 8, 1), (32, 15, 151936, 16, 1), (1, 7, 32000, 4, 0), (2, 4, 2048, 8, 1), (3, 2, 100, 16, 0),
    (64, 2, 3000, 4, 1), (2, 4, 8200, 16, 1),
])
def test_draft_step_workspace_bytes(B, gamma, V, K, dt):
    L = ubt.lib()
    got = L.ubt_draft_step_workspace_bytes(B, gamma, V, K, dt)
    assert got == _step_ws_expected(B, gamma, V, K, 2 if dt == 1 else 4)
    assert got >= 256 + 4 * B * gamma
    assert L.ubt_draft_step_workspace_bytes(0, gamma, V, K, dt) == 0
    assert L.ubt_draft_step_workspace_bytes(B, gamma, K - 1, K, dt) == 0


def _lmh(**kw):
    a = dict(h=FAKE, w=FAKE, M=15, d=2560, V=151936, K=64, ids=FAKE, val=FAKE, lp=None, lse=None, ws=FAKE,
             wsb=1 << 30)
    a.update(kw)
    return ubt.lib().ubt_lm_head_topk(a["h"], a["w"], a["M"], a["d"], a["V"], a["K"], a["ids"], a["val"], a["lp"],
                                      a["lse"], a["ws"], a["wsb"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(h=None), 1), (dict(w=None), 1), (dict(ids=None), 1), (dict(val=None), 1),
    (dict(M=0), 2), (dict(d=48), 2), (dict(d=0), 2), (dict(d=65568), 2), (dict(K=0), 2), (dict(K=65), 2),
    (dict(V=63), 2), (dict(V=2 ** 31), 2),
    (dict(h=ctypes.c_void_p(0x10008)), 4), (dict(w=ctypes.c_void_p(0x10002)), 4),
    (dict(ws=None), 5), (dict(wsb=1000), 5), (dict(ws=ctypes.c_void_p(0x10010)), 5),
])
def test_lm_head_validation(kw, code):
    assert _lmh(**kw) == code


def test_lm_head_workspace_bytes():
    """One (max, sum) and K sorted (key, id) pairs per (row slot, workgroup),
    for 16 row slots per group of rows.  Workgroups: one per compute unit (256 on this GPU
    and when none is visible), at most one per 16-row tile when d is a multiple of 512
    (the k-split kernel), else at most one per 8 tiles."""
    L = ubt.lib()
    al = lambda n: (n + 255) // 256 * 256
    for M, d, V, K in ((15, 2560, 151936, 64), (17, 4096, 151936, 8), (1, 2560, 1000, 1), (3, 96, 1000, 4),
                       (2, 2560, 600, 8)):
        tiles = (V + 15) // 16
        G = min(256, tiles) if d % 512 == 0 else min(256, (tiles + 7) // 8)
        parts = (M + 15) // 16 * G * 16
        assert L.ubt_lm_head_topk_workspace_bytes(M, d, V, K) == al(parts * 8) + al(parts * K * 8)
    assert L.ubt_lm_head_topk_workspace_bytes(0, 2560, 1000, 8) == 0
    assert L.ubt_lm_head_topk_workspace_bytes(4, 2560, 7, 8) == 0
    assert L.ubt_lm_head_topk_workspace_bytes(4, 48, 1000, 8) == 0
    assert L.ubt_lm_head_topk_workspace_bytes(4, 2560, 2 ** 31 - 1, 64) == 0  # the merge's candidates would not fit


def test_lm_head_full_workspace_bytes():
    """The full query is the plain one up to 16 rows where the d-split kernel takes them (d = 512 n
    for n = 2 .. 8 and 10), adds room for the logits of up to 512 rows past that, and rejects what the
    plain one rejects."""
    L = ubt.lib()
    plain, full = L.ubt_lm_head_topk_workspace_bytes, L.ubt_lm_head_topk_full_workspace_bytes
    for d, V, K in ((2560, 151936, 64), (96, 1000, 4), (2880, 50257, 8)):
        assert full(16, d, V, K) == plain(16, d, V, K) if d % 512 == 0 else full(16, d, V, K) >= 16 * V * 4
        assert full(17, d, V, K) >= 17 * V * 4
        assert full(480, d, V, K) >= max(480 * V * 4, plain(480, d, V, K))
        assert full(5000, d, V, K) >= 512 * V * 4
    V, K = 151936, 8
    for d in range(32, 8193, 32):
        split = d % 512 == 0 and d // 512 in (2, 3, 4, 5, 6, 7, 8, 10)
        assert (full(16, d, V, K) == plain(16, d, V, K)) == split, d
        assert split or full(16, d, V, K) >= 16 * V * 4, d
    assert full(0, 2560, 1000, 8) == 0
    assert full(40, 48, 1000, 8) == 0
    assert full(40, 2560, 2 ** 31 - 1, 64) == 0


@pytest.mark.parametrize("d,M,below,above", [
    (2560, 17, 8000, 12000), (2560, 40, 4000, 6000), (2560, 64, 2000, 4000), (2560, 256, 1000, 1500),
    (2560, 480, 600, 800), (4096, 17, 6000, 8000), (4096, 256, 800, 1000),
])
def test_lm_head_few_columns_stay_with_the_row_groups(d, M, below, above):
    """Where the kernel for 16 rows takes d, a head of few columns has no larger workspace to ask for:
    the row groups are faster than the product there (d = 2560, 17 rows of 5,000 columns: 20 us
    against 26).  K = 1, so that the candidates' room does not hide the logits'."""
    L = ubt.lib()
    plain, full = L.ubt_lm_head_topk_workspace_bytes, L.ubt_lm_head_topk_full_workspace_bytes
    assert full(M, d, below, 1) == plain(M, d, below, 1) < M * below * 4
    assert full(M, d, above, 1) >= M * above * 4 > plain(M, d, above, 1)
    assert full(M, d + 32, below, 1) >= M * below * 4  # a d that only the product streams well



def test_tree_attention_workspace_bytes():
    """Partial outputs (D floats) and (max, sum) per query row and part when few workgroups
    would run, nothing when they fill the chip or the context is short; 0 for bad shapes."""
    f = ubt.lib().ubt_tree_attention_workspace_bytes
    n = f(1, 65, 32, 8, 128, 16384)
    assert n > 0 and n % (8 * 65 * 4 * 128 * 4) == (n // (8 * 65 * 4 * 128 * 4 + 8 * 65 * 4 * 8)) * 8 * 65 * 4 * 8
    assert f(32, 65, 32, 8, 128, 4096) == 0
    assert f(1, 65, 32, 8, 128, 256) == 0 and f(1, 65, 32, 8, 128, 0) == 0
    assert f(1, 65, 30, 8, 128, 16384) == 0 and f(1, 300, 32, 8, 128, 16384) == 0 and f(1, 65, 32, 8, 96, 16384) == 0


def test_tree_attention_cut_is_priced():
    """Shapes whose cut measured slower than the whole ranges stay whole (24 and 48 sequences over
    4,096 keys: 176 -> 200 and 343 -> 359 us), and no call asks for more than 256 MiB of scratch,
    however large the cache."""
    f = ubt.lib().ubt_tree_attention_workspace_bytes
    for B, P in ((20, 4096), (24, 4096), (28, 32768), (32, 32768), (48, 4096)):
        assert f(B, 65, 32, 8, 128, P) == 0, (B, P)
    assert f(24, 100, 16, 2, 128, 2048) == 0  # 101 -> 108 us
    for B in (1, 2, 7, 25, 33, 64, 200):
        for N, H, Hkv, D in ((65, 32, 8, 128), (256, 64, 4, 128), (129, 40, 8, 128), (17, 16, 2, 64)):
            for P in (300, 5000, 32768, 131072, 2 ** 31 - 1):
                assert f(B, N, H, Hkv, D, P) <= 257 << 20, (B, N, H, Hkv, D, P)
    assert f(8, 65, 32, 8, 128, 4096) > 0 and f(16, 65, 32, 8, 128, 4096) > 0  # 171 -> 74, 171 -> 121 us


def test_tree_attention_split_workspace_alignment():
    """A misaligned workspace is refused before any launch."""
    bad = ctypes.c_void_p(0x10010)
    assert ubt.lib().ubt_tree_attention_split(FAKE, FAKE, FAKE, FAKE, 1000, FAKE, FAKE, FAKE, FAKE, 2, 17, 4, 2, 64,
                                              ctypes.c_float(0.1), FAKE, 1, None, bad, 1 << 30, None) == 5


def test_cut_sweep_workspace_bytes():
    """Nothing for more than 32 rows and for short rows; the full step query adds it to the
    plain one."""
    L = ubt.lib()
    f = L.ubt_topk_workspace_bytes
    assert f(1, 15, 151936, 64, 1) >= 15 * 8 * (64 * 8 + 8)
    assert f(4, 15, 151936, 64, 1) == 0 and f(1, 15, 50000, 8, 1) == 0
    assert f(1, 15, 63, 64, 1) == 0 and f(1, 65, 151936, 64, 1) == 0
    assert f(1, 15, 72000, 4, 0) == 0 and f(1, 15, 100000, 4, 0) > 0  # fp32: 11.0 -> 11.7, 14.2 -> 12.2 us
    for B, K in ((1, 64), (1, 8), (32, 8)):
        plain = L.ubt_draft_step_workspace_bytes(B, 15, 151936, K, 1)
        assert L.ubt_draft_step_full_workspace_bytes(B, 15, 151936, K, 1) == plain + f(B, 15, 151936, K, 1)
    assert L.ubt_draft_step_full_workspace_bytes(0, 15, 151936, 8, 1) == 0


def test_topk_split_workspace_alignment():
    """A misaligned workspace is refused before any launch."""
    assert ubt.lib().ubt_topk_split(FAKE, 1, 1, 3, 100000, 300000, 100000, 8, FAKE, FAKE, None, None,
                                    ctypes.c_void_p(0x10010), 1 << 20, None) == 5
