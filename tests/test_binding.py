"""The binding's own memory and library calls, without a GPU: the library and the streams are
stand-ins that record what is asked of them."""
from __future__ import annotations

import contextlib

import pytest
import torch

import paper_2609_39972_amd as ubt


class Lib:
    """Every function returns 0, a size query what `sizes` says."""

    def __init__(self, sizes):
        self.sizes, self.calls = sizes, []

    def __getattr__(self, name):
        if not name.startswith("ubt_"):
            raise AttributeError(name)

        def call(*args):
            self.calls.append((name, args))
            return self.sizes.get(name, 0)
        return call

    def names(self):
        return [n for n, _ in self.calls]


class Side:
    """A stream of the caller's, known by its handle only."""
    cuda_stream = 77


@pytest.fixture
def fake(monkeypatch):
    """(library, allocations): allocations holds (bytes, stream handle) of every scratch tensor."""
    lib, made, on = Lib({}), [], [0]

    @contextlib.contextmanager
    def stream(s):
        on.append(s.cuda_stream)
        yield
        on.pop()

    class External:
        def __init__(self, handle, device=None):
            self.cuda_stream = handle

    def workspace(*shape, **kw):
        made.append((shape, on[-1]))
        return torch.zeros(512, dtype=torch.uint8)

    real = torch.empty

    def empty(*a, **kw):
        if kw.get("dtype") == torch.uint8:
            made.append((a, on[-1]))
        return real(*a, **kw)

    monkeypatch.setattr(ubt, "lib", lambda: lib)
    monkeypatch.setattr(ubt, "_need_gpu", lambda *t: None)
    monkeypatch.setattr(ubt, "_stream", lambda s: 0 if s is None else s.cuda_stream)
    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", External)
    monkeypatch.setattr(ubt, "draft_step_workspace", workspace)
    monkeypatch.setattr(ubt, "lm_head_workspace", workspace)
    monkeypatch.setattr(torch, "empty", empty)
    return lib, made


def _bf16(*shape):
    return torch.zeros(*shape, dtype=torch.bfloat16)


@pytest.mark.parametrize("stream,handle", [(None, 0), (Side(), 77)])
def test_draft_step_makes_its_workspace_on_the_calls_stream(fake, stream, handle):
    lib, made = fake
    ubt.draft_step(_bf16(2, 3, 100), _bf16(100, 16), _bf16(100, 16), _bf16(2, 3, 16), torch.zeros(2, dtype=torch.int32),
                   [1.0] * 3, [1.0] * 3, 4, 2, 6, stream=stream)
    assert [s for _, s in made] == [handle]
    assert lib.calls[-1][1][-1] == handle


@pytest.mark.parametrize("stream,handle", [(None, 0), (Side(), 77)])
def test_lm_head_makes_its_workspace_on_the_calls_stream(fake, stream, handle):
    lib, made = fake
    ubt.lm_head_topk(_bf16(20, 64), _bf16(500, 64), 8, stream=stream)
    assert [s for _, s in made] == [handle]
    assert lib.calls[-1][1][-1] == handle


def _attention(**kw):
    B, N, H, Hkv, D, P = 1, 5, 4, 2, 64, 100
    i32 = dict(dtype=torch.int32)
    return ubt.tree_attention(_bf16(B, N, H, D), _bf16(B, P, Hkv, D), _bf16(B, P, Hkv, D), torch.zeros(B, **i32),
                              _bf16(B, N, Hkv, D), _bf16(B, N, Hkv, D), torch.zeros(B, N, 1, **i32),
                              torch.zeros(B, **i32), **kw)


def test_attention_scratch(fake):
    """Scratch of its own only where the call allocates anyway; a workspace is passed on."""
    lib, made = fake
    lib.sizes["ubt_tree_attention_workspace_bytes"] = 4096
    _attention()
    assert [a for a, _ in made] == [(4096,)] and lib.calls[-1][1][-2] == 4096
    _attention(stream=Side())
    assert made[-1] == ((4096,), 77)
    n = len(made)
    given = dict(out=_bf16(1, 5, 4, 64), lse=torch.zeros(1, 5, 4))
    _attention(**given)
    assert len(made) == n and lib.calls[-1][1][-3:-1] == (None, 0)
    ws = torch.zeros(8192, dtype=torch.uint8)
    _attention(workspace=ws, **given)
    assert len(made) == n and lib.calls[-1][1][-3:-1] == (ws.data_ptr(), 8192)
    with pytest.raises(ValueError):
        _attention(workspace=ws[::2], **given)


@pytest.mark.parametrize("rows,dtype", [(1, torch.bfloat16), (15, torch.bfloat16), (15, torch.float32)])
def test_topk_makes_one_call_and_no_scratch(fake, rows, dtype):
    """Few long rows cost the host no size query, allocation or second launch unless the caller
    keeps a workspace, with and without outputs given."""
    lib, made = fake
    lib.sizes["ubt_topk_workspace_bytes"] = 4096
    x = torch.zeros(1, rows, 140000, dtype=dtype)
    out = ubt.topk(x, 64)
    ubt.topk(x, 64, out=out)
    assert lib.names() == ["ubt_topk_split"] * 2 and made == []
    assert lib.calls[-1][1][-3:-1] == (None, 0)
    ws = torch.zeros(4096, dtype=torch.uint8)
    ubt.topk(x, 64, out=out, workspace=ws)
    assert lib.calls[-1][1][-3:-1] == (ws.data_ptr(), 4096) and made == []


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_draft_step_run_allocates_nothing(fake, dtype):
    """Whatever dtype the logits have, and whatever dtype the step was made for."""
    lib, made = fake
    lib.sizes["ubt_topk_workspace_bytes"] = 0
    step = ubt.DraftStep(1, 3, 70000, 8, 4, 8, _bf16(70000, 16), _bf16(70000, 16), _bf16(1, 3, 16),
                         torch.zeros(1, dtype=torch.int32), [1.0] * 3, [1.0] * 3)
    lib.sizes["ubt_topk_workspace_bytes"] = 4096
    n = len(made)
    step.run(torch.zeros(1, 3, 70000, dtype=dtype))
    assert len(made) == n


def test_a_given_step_workspace_keeps_its_old_contract(fake):
    """A caller's workspace may serve calls of other shapes, which leave it alone in ubt_draft_step
    (their counters would lie in another shape's partial results); only a workspace made for the
    call or by DraftStep goes to ubt_draft_step_full."""
    lib, made = fake
    args = (_bf16(2, 3, 100), _bf16(100, 16), _bf16(100, 16), _bf16(2, 3, 16), torch.zeros(2, dtype=torch.int32),
            [1.0] * 3, [1.0] * 3)
    ws = torch.zeros(1024, dtype=torch.uint8)
    ubt.draft_step(*args, 4, 2, 6, workspace=ws)
    assert lib.calls[-1][0] == "ubt_draft_step" and lib.calls[-1][1][-3:-1] == (ws.data_ptr(), 1024)
    assert made == []
    ubt.draft_step(*args, 4, 2, 6)
    assert lib.calls[-1][0] == "ubt_draft_step_full" and len(made) == 1
    step = ubt.DraftStep(2, 3, 100, 4, 2, 6, *args[1:], one_call=True)
    step.run(args[0])
    assert lib.calls[-1][0] == "ubt_draft_step_full" and lib.calls[-1][1][-3] == step.workspace.data_ptr()


def _loss(scales):
    B, gamma, V, K, r = 1, 3, 100, 4, 16
    cand = dict(cand_ids=torch.zeros(B, gamma, K, dtype=torch.int32), cand_logit=torch.zeros(B, gamma, K),
                lse=torch.zeros(B, gamma))
    return ubt.tree_kl_loss(_bf16(B, gamma, V), cand, _bf16(B, gamma, V), torch.zeros(B, gamma, dtype=torch.int32),
                            torch.zeros(B, dtype=torch.int32), _bf16(V, r), _bf16(V, r), _bf16(B, gamma, r), scales,
                            scales)


@pytest.mark.parametrize("scales", [
    [1.0, 0.5, 2.0], (1, 0.5, 2), torch.tensor([1.0, 0.5, 2.0]), torch.tensor([[1.0], [0.5], [2.0]]),
    torch.tensor([1.0, 0.5, 2.0]).numpy(), [torch.tensor(1.0), torch.tensor([0.5]), 2.0], ["1", "0.5", "2"],
], ids=["list", "tuple", "tensor", "column", "numpy", "tensors", "text"])
def test_objective_takes_any_scales(fake, scales):
    """Depth scales in every form that float() converts one by one."""
    lib, _ = fake
    _loss(scales)
    args = lib.calls[-1][1]
    assert [list(a) for a in args if hasattr(a, "_length_")] == [[1.0, 0.5, 2.0]] * 2


@pytest.mark.parametrize("scales", [[1.0, 0.5, 2.0], torch.tensor([1.0, 0.5, 2.0]), ["1", "0.5", "2"]],
                         ids=["list", "tensor", "text"])
def test_step_takes_any_scales(fake, scales):
    lib, _ = fake
    args = (_bf16(2, 3, 100), _bf16(100, 16), _bf16(100, 16), _bf16(2, 3, 16), torch.zeros(2, dtype=torch.int32))
    ubt.draft_step(*args, scales, iter([1.0, 0.5, 2.0]), 4, 2, 6)
    assert [list(a) for a in lib.calls[-1][1] if hasattr(a, "_length_")] == [[1.0, 0.5, 2.0]] * 2
    with pytest.raises(ValueError):
        ubt.draft_step(*args, [1.0, 0.5], scales, 4, 2, 6)


def test_lm_head_workspace_sizes(monkeypatch):
    """The full size by default, the plain one on request."""
    lib = Lib({"ubt_lm_head_topk_full_workspace_bytes": 1 << 20, "ubt_lm_head_topk_workspace_bytes": 1 << 12})
    monkeypatch.setattr(ubt, "lib", lambda: lib)
    real = torch.empty
    made = []

    def empty(n, **kw):
        made.append(n)
        buf = real(n + 256, **kw)
        return buf[-buf.data_ptr() % 256:][:n]

    monkeypatch.setattr(torch, "empty", empty)
    assert ubt.lm_head_workspace(40, 512, 30000, 8, device="cpu").numel() == 1 << 20
    assert ubt.lm_head_workspace(40, 512, 30000, 8, device="cpu", full=False).numel() == 1 << 12
    assert made == [1 << 20, 1 << 12]


@pytest.mark.parametrize("call", ["topk", "lm_head", "step", "attention"])
def test_only_the_workspace_on_the_host(fake, monkeypatch, call):
    """The workspace is looked at, not only the inputs."""
    lib, _ = fake
    ws = torch.zeros(4096, dtype=torch.uint8)

    def need(*ts):
        if any(t is ws for t in ts):
            raise ValueError("host")

    monkeypatch.setattr(ubt, "_need_gpu", need)
    with pytest.raises(ValueError, match="host"):
        if call == "topk":
            ubt.topk(_bf16(1, 2, 100), 4, workspace=ws)
        elif call == "lm_head":
            ubt.lm_head_topk(_bf16(20, 64), _bf16(500, 64), 8, workspace=ws)
        elif call == "step":
            ubt.draft_step(_bf16(2, 3, 100), _bf16(100, 16), _bf16(100, 16), _bf16(2, 3, 16),
                           torch.zeros(2, dtype=torch.int32), [1.0] * 3, [1.0] * 3, 4, 2, 6, workspace=ws)
        else:
            _attention(workspace=ws)
    assert lib.calls == []
