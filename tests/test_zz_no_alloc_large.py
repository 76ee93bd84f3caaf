"""``specdec_step_noalloc`` beyond the small steps (more than 256 logit rows of at
most 16 KB): verification in one launch on the library's completion counts,
eager and replayed from a HIP graph, against ``specdec_step`` bit for bit and
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_22876_amd import workloads as wl
from tests.gpu_util import alloc_outputs, say
from tests.test_zz_no_alloc import _inputs, _one

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["oop", "inplace"])
@pytest.mark.parametrize("dtype,V", [("bf16", 8192), ("f32", 4096), ("f16", 777)])
def test_large_batches_verify_in_one_launch(variant, dtype, V):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2510_22876_amd import specdec as sd
    sd.timing_enable(False)
    w = wl.WORKLOADS["vicuna7b"].scaled(B=70, V=V, L=1, H=2, D=16, logit_dtype=dtype, prompt=("uniform", 16, 120))
    n, W_in, pad_in, cap = wl.initial_geometry(w, 3)
    src0 = wl.make_kv(w, pad_in, W_in, cap, 3, device="cuda")
    pad = torch.as_tensor(np.asarray(pad_in, np.int32), device="cuda")
    inputs = [wl.logits_and_drafts(w, 3, t, device="cuda")[:2] for t in range(3)]
    lg, dr, src = inputs[0][0].clone(), inputs[0][1].clone(), src0.clone()
    dst = src if variant == "inplace" else torch.zeros_like(src)
    o = alloc_outputs(w.B, w.k, w.V, W_in + w.k + 1)

    def step():
        sd.specdec_step_noalloc(lg, dr, pad, W_in, src, dst, o.tokens, o.n_acc, o.bonus, o.pad_out, o.w_new, o.pos,
                                o.mask, o.dev_status)

    def check(t, what):
        say(f"noalloc large {what} {variant} {dtype} inputs={t}")
        e = alloc_outputs(w.B, w.k, w.V, W_in + w.k + 1)
        s = src0.clone()
        d = s if variant == "inplace" else torch.zeros_like(s)
        sd.specdec_step(inputs[t][0], inputs[t][1], pad, W_in, s, d, e.tokens, e.n_acc, e.bonus, e.pad_out, e.w_new,
                        e.pos, e.mask, e.workspace, e.dev_status)
        torch.cuda.synchronize()
        W = int(e.w_new)
        for name in ("tokens", "n_acc", "bonus", "pad_out", "w_new", "dev_status"):
            assert torch.equal(getattr(o, name), getattr(e, name)), (t, name)
        for name in ("pos", "mask"):
            assert torch.equal(getattr(o, name)[:, :W + w.k + 1], getattr(e, name)[:, :W + w.k + 1]), (t, name)
        assert torch.equal(dst[..., :W, :].view(torch.int16), d[..., :W, :].view(torch.int16)), (t, "kv")

    def load(t):
        lg.copy_(inputs[t][0])
        dr.copy_(inputs[t][1])
        src.copy_(src0)
        torch.cuda.synchronize()

    for t in (0, 1, 2, 0):
        load(t)
        step()
        torch.cuda.synchronize()
        check(t, "eager")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for t in (1, 2, 1, 0):
        load(t)
        g.replay()
        torch.cuda.synchronize()
        check(t, "replay")


# Calls on one scratch whose batch size grows and shrinks, so that the counts and
# the lengths of a call lie where an earlier one had others: no draft, the most
# drafts (rows that accept all 64, the prediction past the last draft among
# them), ties, a row out of range, the most rows, one logit a row, and caches
# that are realigned in place by an ordering walk and by chunks.  "small" and
# "long" are calls of the other routes between them.
CONSECUTIVE = {
    "k0": dict(B=300, k=0, V=4096, logit_dtype="f32"),
    "ties": dict(B=52, k=4, V=8191, tie_frac=0.5),
    "bad_row": dict(B=70, k=5, V=3001, bad=(1, 64)),
    "max_k": dict(B=4, k=64, V=777, accept=("list", (64, 0, 63, 64))),
    "small": dict(B=5, k=3, V=4000),
    "most_rows": dict(B=512, k=7, V=65, logit_dtype="f16"),
    "long": dict(B=70, k=5, V=9000),
    "max_k_many": dict(B=63, k=64, V=129, accept=("alternate",), tie_frac=0.1),
    "one_logit": dict(B=2048, k=1, V=1),
    "fewest_rows": dict(B=257, k=0, V=8192, bad=(0,)),
    "ordering_walk": dict(B=52, k=4, V=500, D=128, prompt=("uniform", 20, 700)),
    "chunks": dict(B=70, k=3, V=500, D=128, prompt=("uniform", 20, 700), bad=(7,)),
    "k0_again": dict(B=257, k=0, V=300, tie_frac=0.3, logit_dtype="f32"),
}


@pytest.mark.parametrize("variant", ["oop", "inplace"])
def test_consecutive_calls_of_changing_batch(variant):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2510_22876_amd import specdec as sd
    sd.timing_enable(False)
    for t, name in enumerate([*CONSECUTIVE, *reversed(CONSECUTIVE)]):
        over = dict(L=1, H=2, D=16, logit_dtype="bf16", prompt=("uniform", 8, 60), tie_frac=0.0)
        over.update(CONSECUTIVE[name])
        bad = over.pop("bad", ())
        w = wl.WORKLOADS["vicuna7b"].scaled(**over)
        rows, row_bytes = w.B * (w.k + 1), w.V * (4 if w.logit_dtype == "f32" else 2)
        one_launch = 256 < rows <= 4096 and row_bytes <= 16 * 1024
        assert one_launch == (name not in ("small", "long"))
        say(f"no-alloc call {t}: {name} {variant} B={w.B} k={w.k} V={w.V} {w.logit_dtype}")
        W_in, cap, pad, logits, draft, src, s_rows = _inputs(w, seed=60 + t)
        pad = pad.copy()
        pad[list(bad)] = W_in - w.k                    # outside [0, W_in - (k + 1)]
        inp = (W_in, cap, pad, logits, draft, src, s_rows)
        got = _one(sd, w, *inp, variant, noalloc=True)
        ref = _one(sd, w, *inp, variant, noalloc=False)
        for key in ref:
            assert np.array_equal(np.asarray(ref[key]), np.asarray(got[key])), (t, name, key)
        assert int(got["dev_status"][0]) == (sd.DEV_BAD_PAD_IN | sd.DEV_BAD_PAD_OUT if bad else 0)
        good = [i for i in range(w.B) if i not in bad]
        v = oracle.verify(logits[good].cpu(), w.logit_dtype, draft[good].cpu().numpy(), pad[good], W_in)
        for key in ("tokens", "n_acc", "bonus", "pad_out"):
            assert np.array_equal(got[key][good], v[key]), (t, name, key)
        assert int(got["w_new"][0]) == v["w_new"] and (got["pad_out"][list(bad)] == -1).all()
        if name == "max_k":
            assert got["n_acc"].tolist() == [64, 0, 63, 64]
