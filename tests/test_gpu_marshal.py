"""The native argument marshalling against the Python marshalling of the same
wrappers: the same outputs, the same returned width and the same exceptions for
arguments that either refuses."""
import numpy as np
import pytest
import torch

from paper_2510_22876_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2510_22876_amd import specdec
    assert specdec._native is not None, "the native marshalling is not built"
    return specdec


def _calls(sd, dtype):
    """{name: (call, outputs)} on fresh buffers, equal from call to call."""
    w = wl.WORKLOADS["tiny"].scaled(B=3, logit_dtype=dtype, extra_cap=5)
    n, W_in, pad, cap = wl.initial_geometry(w, 3)
    logits, draft, *_ = wl.logits_and_drafts(w, 3, device="cuda")
    sl, dl, sdraft, ua, us = wl.sampled_inputs(w, 3, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    pad = torch.as_tensor(pad, device="cuda")

    def buffers():
        b = sd.StepBuffers(w.B, w.k, w.V, W_in + w.k + 1)
        for t in (b.tokens, b.n_acc, b.bonus, b.pad_out, b.w_new, b.pos, b.mask):
            t.fill_(7)
        src = wl.make_kv(w, pad.cpu().numpy(), W_in, cap, 3, device="cuda")
        s = wl.make_token_rows(w, pad.cpu().numpy(), W_in, cap + 1, 3, -1, device="cuda")
        return b, src, torch.zeros_like(src), s, torch.zeros_like(s)

    def step(noalloc=False, sampled=False, **kw):
        b, src, dst, s_in, s_out = buffers()
        out = (b.tokens, b.n_acc, b.bonus, b.pad_out, b.w_new, b.pos, b.mask)
        kw = dict(s_in=s_in, s_out=s_out, pad_id=-1, dev_status=b.dev_status, sync_w_new=True, **kw)
        if sampled:
            ws = sd.alloc_sample_workspace(w.B, w.k, w.V)
            r = sd.specdec_step_sample(sl, dl, sdraft, pad, ua, us, 1.0, W_in, src, dst, *out, ws, **kw)
        elif noalloc:
            r = sd.specdec_step_noalloc(logits, draft, pad, W_in, src, dst, *out, **kw)
        else:
            r = sd.specdec_step(logits, draft, pad, W_in, src, dst, *out, b.workspace, **kw)
        return (r, *out, dst, s_out, b.dev_status)

    def verify(sampled=False, bonus=True, stream=None):
        b = buffers()[0]
        out = (b.tokens, b.n_acc, b.bonus if bonus else None, b.pad_out, b.w_new)
        if sampled:
            r = sd.specdec_verify_sample(sl, dl, sdraft, pad, ua, us, 1.0, W_in, *out,
                                         sd.alloc_sample_workspace(w.B, w.k, w.V), b.dev_status, stream)
        else:
            r = sd.specdec_verify_greedy(logits, draft, pad, W_in, *out, b.workspace, stream=stream)
        return (r, *out, b.dev_status)

    def pool(gather):
        lens = np.array([9, 20, 14, 3, 11], np.int32)
        kv, tok = wl.make_pool(w, lens, 40, 41, 3, device="cuda")
        lens, slots = torch.as_tensor(lens, device="cuda"), torch.tensor([3, 1, 4], **i32)
        batch = torch.zeros((w.L, 2, 3, w.H, 20 + w.k + 1, w.D), dtype=torch.bfloat16, device="cuda")
        btok, pads = torch.zeros((3, 20 + w.k + 2), **i32), torch.zeros(3, **i32)
        pos = torch.zeros((3, 20 + w.k + 1), dtype=torch.int64, device="cuda")
        mask = torch.zeros_like(pos, dtype=torch.uint8)
        r = sd.specdec_gather_batch(kv, tok, lens, slots, 20, batch, pads, btok, pos, mask, w.k, -1)
        if not gather:
            n_acc = torch.tensor([0, 4, 2], **i32)
            tokens = torch.arange(3 * (w.k + 1), **i32).view(3, w.k + 1)
            r = sd.specdec_scatter_accepted(batch, pads, tokens, n_acc, slots, 20, kv, tok, lens, btok,
                                            sd.WRITEBACK_APPEND)
        return (r, kv, tok, lens, batch, btok, pads, pos, mask)

    def varlen(pos=True):
        cu = torch.tensor([0, 9, 15, 40], **i32)
        src = torch.randn((2, 2, 40, 2, 16), generator=torch.Generator("cuda").manual_seed(1), device="cuda").bfloat16()
        dst, cu_out = torch.zeros_like(src), torch.zeros(4, **i32)
        p = torch.zeros(40, dtype=torch.int64, device="cuda") if pos else None
        r = sd.specdec_varlen_rollback(src, dst, cu, torch.tensor([1, 0, 3], **i32), 3, 25, cu_out, p)
        return (r, dst, cu_out, p)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    return {"step": step, "noalloc": lambda: step(noalloc=True), "sampled": lambda: step(sampled=True),
            "verify": verify, "verify_stream": lambda: verify(stream=side), "verify_no_bonus": lambda: verify(bonus=False),
            "verify_sample": lambda: verify(sampled=True), "gather": lambda: pool(True), "scatter": lambda: pool(False),
            "varlen": varlen, "varlen_no_pos": lambda: varlen(pos=False)}


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_native_and_python_marshalling_agree(sd, monkeypatch, dtype):
    calls = _calls(sd, dtype)
    native = {}
    for name, f in calls.items():
        native[name] = f()
        torch.cuda.synchronize()
    monkeypatch.setattr(sd, "_native", None)
    for name, f in calls.items():
        want = f()
        torch.cuda.synchronize()
        for a, b in zip(native[name], want):
            assert torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b, f"{name}: outputs differ"


def test_refused_arguments_raise_alike(sd, monkeypatch):
    w = wl.WORKLOADS["tiny"]
    logits, draft, *_ = wl.logits_and_drafts(w, 0, device="cuda")
    b = sd.StepBuffers(w.B, w.k, w.V, 80)
    pad = torch.zeros(w.B, dtype=torch.int32, device="cuda")
    good = dict(logits=logits, draft=draft, pad_in=pad, W_in=64, tokens=b.tokens, n_acc=b.n_acc, bonus=b.bonus,
                pad_out=b.pad_out, w_new=b.w_new, workspace=b.workspace)
    wrong = [dict(draft=draft.long()), dict(draft=draft.cpu()), dict(pad_in=pad[:1]), dict(logits=logits[..., ::2]),
             dict(logits=logits.double()), dict(n_acc=None), dict(workspace=b.workspace[:1]), dict(W_in=2), dict(W_in=6.5),
             dict(pad_out=pad), dict(tokens=b.tokens.t()), dict(w_new=b.n_acc), dict(stream="main")]

    def outcome(change):
        try:
            sd.specdec_verify_greedy(**{**good, **change})
        except Exception as e:
            return type(e), str(e)
        return None

    native = [outcome(c) for c in wrong]
    assert outcome({}) is None
    monkeypatch.setattr(sd, "_native", None)
    assert native == [outcome(c) for c in wrong] and all(native)
    torch.cuda.synchronize()
